// Point splatting of per-octant arrays into novel views (Sec. 3.3): every
// fragment is projected, covers a k x k pixel square (at least one pixel),
// and per pixel the nearest fragment wins, as in deferred shading.
//
// Screen-tile ownership: every view is cut into tiles of 64 x 64 pixels and
// one workgroup owns a tile, holding its depth test in LDS, so no z-buffer
// entry is touched by more than one workgroup and no global atomic decides a
// pixel. The arrays are cut into chunks of 64 consecutive fragments (one per
// lane); in Morton order a chunk is a compact piece of surface, and so is a
// run of 64 consecutive chunks, and of 64 such runs, and so on: the bounding
// boxes of those runs form a tree over the arrays that a tile's workgroup
// walks to find the few chunks that can reach it, with no binning pass and
// no atomic on global memory.
//
//   k_chunk_box   a workgroup per group of 64 chunks: the bounding boxes of
//                 the chunks' fragment positions and of the group (and the
//                 ranges of scenes their keys belong to), packed positions
//   k_node_box    one wave per node of the next level up: the union of its
//                 64 children's boxes, up to a level of at most 512 nodes
//   k_tile_est    a wave per tile: the tree walked down to the groups of
//                 chunks that can reach the tile, which set how many
//                 workgroups draw it (a busy tile is split into up to 16
//                 sub-tiles) and the order of the draw: items listed in 8
//                 classes of their share of groups, busiest first
//   k_tile_splat  one workgroup of 16 waves per tile or sub-tile: z-tile of 64-bit keys
//                 (fp32 depth bits << 32 | fragment index) in LDS, cleared;
//                 the tree walked from its top level, a node's 64 children
//                 tested at once (one per lane) by projecting the child's box
//                 into the view with a margin that covers the fp32 rounding
//                 of every fragment inside it; every chunk that can reach the
//                 tile projected fragment by fragment (fp32 3x4 transform
//                 without fused multiply-adds) with an LDS 64-bit minimum for
//                 each footprint pixel inside the (sub-)tile; then each pixel
//                 of it written once: key, winner's colour (w1), depth and
//                 coverage
//
// A batch (many scenes in one key space, key = scene << 3L | Morton code)
// runs the same kernels over (scene, view) slots; a fragment only draws into
// the views of its own scene, and the matrices are read from device memory.
#include <math.h>
#include <string.h>

#include "fhv_common.h"

namespace fhv {

namespace {

constexpr int kChunk = kWave;       // fragments per chunk, one per lane
constexpr int kTile = 64;           // tile side in pixels
constexpr int kTilePix = kTile * kTile;

// What every kernel needs to know about the call.
struct TileArgs {
    uint32_t n_scenes;     // 1 for fhv_splat
    uint32_t scenes;       // a batch: the boxes have scene ranges
    uint32_t n_views;      // views per scene
    uint32_t width, height;
    uint32_t nx, ny;       // tiles per row and per column of a view
    uint32_t per_view;     // nx * ny
    uint32_t n_tiles;      // n_scenes * n_views * per_view
    uint32_t shift;        // batches: scene = key >> shift; else 64 (no scene bits)
    uint32_t cap_w;        // PPFL capture width (pixel keys)
    uint64_t cap_frag, cap_occ;
    // chunk tree for cap_frag fragments: levels (0 chunks, the last one the
    // level of at most kTopNodes nodes), where each level's boxes start (in
    // nodes), nodes of all levels
    uint32_t levels;
    uint64_t lv_off[8];
    float span[3];         // bound of the positions' coordinates
    float unit[3];         // of the boxes, in positions
    float inset;           // of z positions from the ends of their units (x, y: 1/2)
    uint32_t qs;           // POFL: log2 of it
    uint64_t n_nodes;
    uint32_t gbits;        // POFL: bits per grid coordinate (octree depth + 8)
};

// Matrix, footprint side and offset 1/2 - k/2 of view slot g (scene g / V,
// view g % V): from the kernel arguments (one scene) or, for a batch, from
// device memory [scene][view][12] with one footprint for all views.
template <bool kBatch>
struct ViewSrc {
    const ViewArgs& va;
    const float* vm;
    __device__ __forceinline__ const float* m(uint32_t g) const
    {
        return kBatch ? vm + 12ull * g : va.m[g];
    }
    __device__ __forceinline__ uint32_t k(uint32_t g) const { return kBatch ? va.k[0] : va.k[g]; }
    __device__ __forceinline__ float c(uint32_t g) const { return kBatch ? va.c[0] : va.c[g]; }
};

__device__ __forceinline__ uint64_t frag_total(const uint64_t* n_frag, uint64_t cap)
{
    const uint64_t nf = *n_frag;
    return nf < cap ? nf : cap;
}

// The chunk tree: level 0 holds the chunks' boxes, every node of level
// l + 1 the union of the boxes of its kFan children (nodes kFan n .. kFan n
// + kFan - 1 of level l), up to a level of few nodes.
constexpr int kFan = kWave;
constexpr uint32_t kCounterStep = 32;   // of the item counters: lines of their own

// Nodes of level l for F fragments.
__device__ __forceinline__ uint64_t level_count(uint64_t F, uint32_t l)
{
    const uint32_t sh = 6 * (l + 1);   // kChunk and kFan are 2^6
    return (F + ((uint64_t)1 << sh) - 1) >> sh;
}

// The level the tiles' walks start from, all of whose nodes they test: the
// lowest (of level 1 and up) with at most kTopNodes nodes. Each level above
// would be one more step of loads and barriers for every tile.
constexpr uint32_t kTopNodes = 512;

__host__ __device__ __forceinline__ uint32_t top_level(uint64_t F)
{
    uint32_t l = 1;
    while (((F + ((uint64_t)1 << (6 * (l + 1))) - 1) >> (6 * (l + 1))) > kTopNodes) ++l;
    return l;
}

// Integer position of a fragment in the view's input space: PPFL pixel x, y
// and depth24, POFL grid x, y, z (the views take x + 1/2 and so on, but PPFL
// depths as they are). Pixel keys stay below 2^28, octant keys of depth 10
// and less below 2^30.
struct Pos3 {
    uint32_t x, y, z;
};

template <int kMode>
__device__ __forceinline__ Pos3 frag_pos(uint32_t w0, uint64_t key, const TileArgs& ta)
{
    if (kMode == FHV_PPFL) {
        const uint32_t k = (uint32_t)key, y = k / ta.cap_w;
        return Pos3{k - y * ta.cap_w, y, w0 & 0xFFFFFFu};
    }
    uint32_t kx, ky, kz;
    if (ta.gbits <= 18) {
        const uint32_t k = (uint32_t)key;
        kx = compact3_10(k >> 2);
        ky = compact3_10(k >> 1);
        kz = compact3_10(k);
    } else {
        kx = compact3(key >> 2);
        ky = compact3(key >> 1);
        kz = compact3(key);
    }
    return Pos3{(kx << 8) | (w0 & 0xFFu), (ky << 8) | ((w0 >> 8) & 0xFFu), (kz << 8) | ((w0 >> 16) & 0xFFu)};
}

// Packed position of a fragment for the tile kernel: bit 63 set when the
// fragment is drawn at all; POFL: grid x, y, z (gbits each) and the scene
// above them; PPFL: pixel x, y (14 bits each) and depth24.
template <int kMode>
__device__ __forceinline__ uint64_t pack_pos(const Pos3& p, uint32_t scene, bool ok, const TileArgs& ta)
{
    if (!ok) return 0;
    if (kMode == FHV_PPFL) return (1ull << 63) | p.x | ((uint64_t)p.y << 14) | ((uint64_t)p.z << 28);
    const uint32_t S = ta.gbits;
    return (1ull << 63) | p.x | ((uint64_t)p.y << S) | ((uint64_t)p.z << (2 * S)) | ((uint64_t)scene << (3 * S));
}

// A node's box in memory: one uint4 (units: ta.unit), and for a batch a
// second one with the range of scenes in x, y.
template <bool kBatch>
constexpr uint32_t kNodeWords = kBatch ? 2 : 1;   // uint4 per node

struct NodeBox {
    BoxMin b;
    uint32_t s0, s1;
};

__device__ __forceinline__ NodeBox node_none() { return NodeBox{BoxMin{{~0u, ~0u, ~0u}}, ~0u, 0u}; }

template <bool kBatch>
__device__ __forceinline__ NodeBox node_join(const NodeBox& a, const NodeBox& b)
{
    NodeBox o{box_join(a.b, b.b), 0u, 0u};
    if (kBatch) {
        o.s0 = a.s0 < b.s0 ? a.s0 : b.s0;
        o.s1 = a.s1 > b.s1 ? a.s1 : b.s1;
    }
    return o;
}

template <bool kBatch>
__device__ __forceinline__ void node_store(uint4* p, const NodeBox& n)
{
    p[0] = box_store(n.b);
    if (kBatch) p[1] = make_uint4(n.s0, n.s1, 0u, 0u);
}

// One workgroup of 8 waves per group of 64 chunks, four chunks of a wave at
// a time with all their loads in flight: the chunks' boxes, the group's, and
// every fragment's packed position. Bound by the 16 bytes of record read and
// 8 of position written per fragment; a box takes three register reductions
// of two 16-bit values (as butterflies of eight 32-bit values through LDS
// permutes they bound the kernel: 5.2 M fragments 52 us, 45 M 447 us, and
// the groups' boxes took a launch of their own; here 31 and 267 us).
constexpr int kBoxWaves = 8;

template <int kMode, bool kBatch>
__global__ void __launch_bounds__(kBoxWaves * kWave)
k_chunk_box(const uint4* __restrict__ frag, const uint64_t* __restrict__ oct_key, const uint64_t* __restrict__ n_frag,
            TileArgs ta, uint4* __restrict__ box, uint64_t* __restrict__ pos, uint32_t* __restrict__ bucket)
{
    __shared__ NodeBox part[kBoxWaves];
    if (blockIdx.x == 0 && threadIdx.x < 9) bucket[threadIdx.x * kCounterStep] = 0;   // the tile pass's item counters, anew
    if (ta.cap_occ == 0) return;   // no table rows: nothing to draw
    const uint64_t F = frag_total(n_frag, ta.cap_frag);
    const uint64_t nch = (F + kChunk - 1) / kChunk, ngr = (nch + kFan - 1) / kFan;
    const int lane = __lane_id();
    const uint32_t wv = uniform32(threadIdx.x / kWave);
    const uint64_t kmask = ta.shift >= 64 ? ~0ull : (1ull << ta.shift) - 1ull;
    constexpr uint32_t kPer = kFan / kBoxWaves;
    constexpr int kU = 4;
    for (uint64_t g = blockIdx.x; g < ngr; g += gridDim.x) {
        NodeBox all = node_none();
        for (uint32_t k0 = 0; k0 < kPer; k0 += kU) {
            const uint64_t ch = g * kFan + wv * kPer + k0;
            if (ch >= nch) break;   // wave-uniform
            uint4 r[kU];
            uint64_t key[kU];
            bool ok[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint64_t f = (ch + u) * kChunk + lane;
                ok[u] = f < F;
                r[u] = frag[ok[u] ? f : 0];
                ok[u] = ok[u] && r[u].w < ta.cap_occ;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) key[u] = oct_key[ok[u] ? r[u].w : 0];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                if (ch + u >= nch) continue;   // wave-uniform
                const uint32_t scene = kBatch ? (uint32_t)(key[u] >> ta.shift) : 0u;
                const bool in = ok[u] && (!kBatch || scene < ta.n_scenes);
                const Pos3 p = frag_pos<kMode>(r[u].x, key[u] & kmask, ta);
                pos[(ch + u) * kChunk + lane] = pack_pos<kMode>(p, scene, in, ta);
                const uint32_t sxy = kMode == FHV_PPFL ? 0u : ta.qs, sz = kMode == FHV_PPFL ? 8u : ta.qs;
                NodeBox n{wave_box(p.x >> sxy, p.y >> sxy, p.z >> sz, in), 0u, 0u};
                if (kBatch) {
                    n.s0 = ~wave_all_max(in ? ~scene : 0u);
                    n.s1 = wave_all_max(in ? scene : 0u);
                }
                if (lane == 0) node_store<kBatch>(box + kNodeWords<kBatch> * (ch + u), n);
                all = node_join<kBatch>(all, n);
            }
        }
        if (lane == 0) part[wv] = all;
        __syncthreads();
        if (threadIdx.x == 0) {
            NodeBox n = part[0];
            for (int w = 1; w < kBoxWaves; ++w) n = node_join<kBatch>(n, part[w]);
            node_store<kBatch>(box + kNodeWords<kBatch> * (ta.lv_off[1] + g), n);
        }
        __syncthreads();
    }
}

// Boxes of level l >= 2: one wave per node, one lane per child.
template <bool kBatch>
__global__ void __launch_bounds__(kBlock)
k_node_box(const uint64_t* __restrict__ n_frag, TileArgs ta, uint32_t l, uint4* __restrict__ box)
{
    if (ta.cap_occ == 0) return;
    const uint64_t F = frag_total(n_frag, ta.cap_frag);
    const uint64_t n = level_count(F, l), nc = level_count(F, l - 1);
    const uint64_t n_waves = (uint64_t)gridDim.x * (kBlock / kWave);
    for (uint64_t node = uniform64((uint64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave); node < n;
         node += n_waves) {
        const uint64_t c = node * kFan + __lane_id();
        NodeBox b = node_none();
        if (c < nc) {
            const uint4* p = box + kNodeWords<kBatch> * (ta.lv_off[l - 1] + c);
            b.b = box_load(p[0]);
            if (kBatch) {
                b.s0 = p[1].x;
                b.s1 = p[1].y;
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) b.b.v[k] = wave_pk_min(b.b.v[k]);
        if (kBatch) {
            b.s0 = ~wave_all_max(~b.s0);
            b.s1 = wave_all_max(b.s1);
        }
        if (__lane_id() == 0) node_store<kBatch>(box + kNodeWords<kBatch> * (ta.lv_off[l] + node), b);
    }
}

// Workgroup order: consecutive workgroups go to the 8 accelerator dies in
// turn, so that the tiles of one die form one contiguous run of tile indices
// (neighbouring tiles share chunks, which then meet in that die's cache).
__device__ __forceinline__ uint32_t die_major(uint32_t b, uint32_t n)
{
    const uint32_t q = n / 8, r = n % 8, x = b % 8, j = b / 8;
    return x < r ? x * (q + 1) + j : r * (q + 1) + (x - r) * q + j;
}

constexpr int kTileWaves = 16;                 // waves per tile workgroup
constexpr int kTileThreads = kTileWaves * kWave;
constexpr uint32_t kFront = 2048;              // breadth-first frontier capacity (node ids)
// Ordering and splitting the tiles: a tile whose walk reaches n groups of
// chunks is drawn by P workgroups, ceil(n / kSplitGroups) rounded up to a
// power of two (at most kMaxParts), each on a sub-tile of 64 x 64 / P
// pixels (square or twice as wide as tall: fewer chunks straddle two
// sub-tiles than narrow column strips), with at most kMaxItems workgroups beyond one per tile per launch; the workgroups
// start in decreasing order of their share of groups (8 classes), the
// busiest first. Launches of 2^22 tiles or more keep one workgroup per tile
// in the plain order.
constexpr uint32_t kSplitGroups = 64, kMaxParts = 16, kMaxItems = 4096, kOrderTiles = 1u << 22;
constexpr uint32_t kEstWaves = 16;             // waves (tiles) per workgroup of the estimate pass
// A tile whose walk ends on at most kGroupList groups of chunks gets them
// listed by the estimate pass, and its workgroup in the tile pass starts
// from that list instead of walking the tree again.
constexpr uint32_t kGroupList = 32;

// What one tile's workgroup knows about its view.
struct TileView {
    float M[12];
    float c;
    float mg[3];      // margins of a box's extent along the matrix rows (box_reaches)
    int32_t k;
    uint32_t scene;
    int32_t X0, Y0;
    int32_t XS, XE;   // the sub-tile this workgroup draws: columns [XS, XE),
    int32_t YS, YE;   // rows [YS, YE), within the tile
    float fxs, fxe, fys, fye;   // the same, as far as the image goes
};

// Workgroups beyond one per tile: up to kMaxItems; none when the tiles are
// not ordered.
__host__ __device__ __forceinline__ uint32_t split_items(uint32_t n_tiles)
{
    if (n_tiles >= kOrderTiles) return 0;
    const uint32_t m = 2 * ((n_tiles + 7) / 8 * 8);
    return m < kMaxItems ? m : kMaxItems;
}

// Whether a fragment in the box at b can reach the (sub-)tile: its footprint
// starts at floor(s + c) and is k pixels wide per axis, so columns [XS, XE)
// are reached where XS - k + 1 <= s + c < XE, and fragments with depth <= 0
// are not drawn. Each row of the matrix over the box lies within the value
// at its centre plus and minus the absolute row times its half sides, widened
// by 2^-20 of the sum of absolute terms over the whole input space: a
// fragment's fp32 projection is off by less than 0.4 of that, the extent's
// own rounding by less than 0.5. Written so that values that are not numbers
// reject nothing.
template <bool kBatch>
__device__ __forceinline__ bool box_reaches(const uint4* __restrict__ b, const TileArgs& ta, const TileView& tv)
{
    const uint4 v = b[0];
    const uint32_t lx = v.x & 0xFFFFu, ly = v.x >> 16, lz = v.y & 0xFFFFu, ux = v.y >> 16, uy = v.z & 0xFFFFu,
                   uz = v.z >> 16;
    bool ok = lx <= ux;   // some drawable fragment
    if (kBatch) ok = ok && b[1].x <= tv.scene && tv.scene <= b[1].y;
    // the box's units reach from their lowest position to the next unit's, and
    // positions lie half a step from both: without it a box that ends on a
    // plane of the octree met the tile behind the plane, and of a view whose
    // tiles' borders are such planes up to 1.6 times as many nodes were walked
    // (tile pass of 67.6 M fragments in one 64 x 64 view 11.3 ms, here 8.3)
    const float wx = 0.5f * ta.unit[0], wy = 0.5f * ta.unit[1], wz = 0.5f * ta.unit[2];
    const float cx = (float)(lx + ux + 1) * wx, cy = (float)(ly + uy + 1) * wy, cz = (float)(lz + uz + 1) * wz;
    const float hx = __builtin_fmaf((float)(ux - lx + 1), wx, -0.5f), hy = __builtin_fmaf((float)(uy - ly + 1), wy, -0.5f),
                hz = __builtin_fmaf((float)(uz - lz + 1), wz, -ta.inset);
    float s[3], e[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const float* m = tv.M + 4 * r;
        s[r] = __builtin_fmaf(m[0], cx, __builtin_fmaf(m[1], cy, __builtin_fmaf(m[2], cz, m[3])));
        e[r] = __builtin_fmaf(fabsf(m[0]), hx, __builtin_fmaf(fabsf(m[1]), hy, __builtin_fmaf(fabsf(m[2]), hz, tv.mg[r])));
    }
    const float x = s[0] + tv.c, y = s[1] + tv.c;
    return ok && !(x - e[0] >= (float)tv.XE) && !(x + e[0] < (float)(tv.XS - tv.k + 1)) &&
           !(y - e[1] >= (float)tv.YE) && !(y + e[1] < (float)(tv.YS - tv.k + 1)) && !(s[2] + e[2] <= 0.0f);
}

// Which of the kFan children of node `node` (on level l, children on level
// l - 1 with n nodes) can reach the tile: a bit per lane.
template <bool kBatch>
__device__ __forceinline__ uint64_t test_children(const uint4* __restrict__ box, const TileArgs& ta, uint64_t n,
                                                  uint32_t l, uint32_t node, const TileView& tv)
{
    const uint64_t c = (uint64_t)node * kFan + __lane_id();
    return __ballot(c < n && box_reaches<kBatch>(box + kNodeWords<kBatch> * (ta.lv_off[l - 1] + (c < n ? c : 0)), ta, tv));
}

// The lanes' fragments (packed position p, array index f) drawn into the
// z-tile. The vector unit is what the tile pass keeps busiest (two thirds of
// the time), most of it here: positions are taken apart by 32-bit extracts
// (64-bit shifts take several cycles each; depths below 8, whose z starts in
// the low word, keep them), and a pixel is tested in floating point against
// the tile's part within the image, whose borders are exact in it, which
// also drops what is not a number (three 1080p views 97 -> 91 us, a 4K pair
// 475 -> 454).
template <int kMode, bool kBatch>
__device__ __forceinline__ void draw_pos(uint64_t p, uint32_t f, const TileArgs& ta, const TileView& tv,
                                         unsigned long long* zt)
{
    const uint32_t lo = (uint32_t)p, hi = (uint32_t)(p >> 32);
    bool ok = (int32_t)hi < 0;
    float x, y, z;
    if (kMode == FHV_PPFL) {
        x = (float)(lo & 0x3FFFu) + 0.5f;
        y = (float)((lo >> 14) & 0x3FFFu) + 0.5f;
        z = (float)(__builtin_amdgcn_alignbit(hi, lo, 28) & 0xFFFFFFu);
    } else {
        const uint32_t S = ta.gbits, gm = (1u << S) - 1u;
        uint32_t iz, sc;
        if (S >= 16) {   // uniform
            iz = (hi >> (2 * S - 32)) & gm;
            sc = (hi & 0x7FFFFFFFu) >> (3 * S - 32);
        } else {
            iz = (uint32_t)(p >> (2 * S)) & gm;
            sc = (uint32_t)((p & ~(1ull << 63)) >> (3 * S));
        }
        x = (float)(lo & gm) + 0.5f;
        y = (float)(__builtin_amdgcn_alignbit(hi, lo, S) & gm) + 0.5f;
        z = (float)iz + 0.5f;
        if (kBatch) ok = ok && sc == tv.scene;
    }
    const float* M = tv.M;
    const float sx = ((M[0] * x + M[1] * y) + M[2] * z) + M[3];
    const float sy = ((M[4] * x + M[5] * y) + M[6] * z) + M[7];
    const float d = ((M[8] * x + M[9] * y) + M[10] * z) + M[11];
    const float fx = floorf(sx + tv.c), fy = floorf(sy + tv.c);
    const unsigned long long zk = ((unsigned long long)__float_as_uint(d) << 32) | (unsigned long long)f;
    const int32_t k = tv.k, X0 = tv.X0, Y0 = tv.Y0;
    if (k == 1) {
        if (ok && d > 0.0f && fx >= tv.fxs && fx < tv.fxe && fy >= tv.fys && fy < tv.fye)
            atomicMin(zt + ((int32_t)fy - Y0) * kTile + ((int32_t)fx - X0), zk);
        return;
    }
    // (fx + k is exact wherever it can lie within the tile)
    const float fk = (float)k, xa = fx > tv.fxs ? fx : tv.fxs, xb = fx + fk < tv.fxe ? fx + fk : tv.fxe;
    const float ya = fy > tv.fys ? fy : tv.fys, yb = fy + fk < tv.fye ? fy + fk : tv.fye;
    if (!(ok && d > 0.0f && xa < xb && ya < yb && fx == fx && fy == fy)) return;
    const int32_t ixa = (int32_t)xa - X0, ixb = (int32_t)xb - X0, iyb = (int32_t)yb - Y0;
    for (int32_t yy = (int32_t)ya - Y0; yy < iyb; ++yy)
        for (int32_t xx = ixa; xx < ixb; ++xx) atomicMin(zt + yy * kTile + xx, zk);
}

// The chunks q[i] (or base + i when q is null), i = i0, i0 + step, ... < n,
// drawn in batches of kDrawBatch, the next batch's positions loading while
// the current batch is drawn (so that up to 2 kDrawBatch loads of a wave
// are in flight). Chunks beyond the arrays' end hold positions that are not
// drawn.
constexpr int kDrawBatch = 4;

template <int kMode, bool kBatch>
__device__ __forceinline__ void draw_queue(const uint32_t* q, uint64_t base, uint32_t i0, uint32_t step, uint32_t n,
                                           const uint64_t* __restrict__ pos, const TileArgs& ta, const TileView& tv,
                                           unsigned long long* zt)
{
    if (i0 >= n) return;
    const int lane = __lane_id();
    // chunk ids fit 32 bits (fewer than 2^32 chunks per launch). Past the end the
    // last chunk is loaded again (and not drawn): loads under branches made the
    // wait before a draw one for all of them, the next batch's too (tile pass
    // of 48.8 M fragments in one 64 x 64 view 5.27 ms, here 4.48).
    auto chunk = [&](uint32_t i) -> uint32_t {
        const uint32_t k = i < n ? i : n - 1;
        return q ? q[k] : (uint32_t)base + k;
    };
    uint32_t ca[kDrawBatch];
    uint64_t pa[kDrawBatch];
#pragma unroll
    for (int j = 0; j < kDrawBatch; ++j) ca[j] = chunk(i0 + (uint32_t)j * step);
#pragma unroll
    for (int j = 0; j < kDrawBatch; ++j) pa[j] = pos[(uint64_t)ca[j] * kChunk + lane];
    for (uint32_t ib = i0; ib < n; ib += kDrawBatch * step) {
        uint32_t cb[kDrawBatch];
        uint64_t pb[kDrawBatch];
#pragma unroll
        for (int j = 0; j < kDrawBatch; ++j) cb[j] = chunk(ib + (uint32_t)(kDrawBatch + j) * step);
#pragma unroll
        for (int j = 0; j < kDrawBatch; ++j) pb[j] = pos[(uint64_t)cb[j] * kChunk + lane];
#pragma unroll
        for (int j = 0; j < kDrawBatch; ++j)
            if (ib + (uint32_t)j * step < n)
                draw_pos<kMode, kBatch>(pa[j], ca[j] * kChunk + (uint32_t)lane, ta, tv, zt);
#pragma unroll
        for (int j = 0; j < kDrawBatch; ++j) {
            ca[j] = cb[j];
            pa[j] = pb[j];
        }
    }
}

// The view of tile `tile` (slot g = tile / per_view) for the walk and the draw.
template <bool kBatch>
__device__ __forceinline__ TileView tile_view(uint32_t tile, const TileArgs& ta, const ViewArgs& va, const float* vm,
                                              bool drawn, uint32_t part = 0, uint32_t n_parts = 1)
{
    const uint32_t g = tile / ta.per_view, t = tile % ta.per_view;
    TileView tv;
    tv.X0 = (int32_t)((t % ta.nx) * kTile);
    tv.Y0 = (int32_t)((t / ta.nx) * kTile);
    // n_parts (a power of two up to 16) square or 2:1 sub-tiles: 2 x 1,
    // 2 x 2, 4 x 2, 4 x 4 (columns x rows), numbered along the rows
    const uint32_t lg = 31u - (uint32_t)__builtin_clz(n_parts | 1u);
    const uint32_t cols = 1u << ((lg + 1) >> 1), rows = n_parts >> ((lg + 1) >> 1);
    tv.XS = tv.X0 + (int32_t)((part % cols) * (kTile / cols));
    tv.XE = tv.XS + (int32_t)(kTile / cols);
    tv.YS = tv.Y0 + (int32_t)((part / cols) * (kTile / rows));
    tv.YE = tv.YS + (int32_t)(kTile / rows);
    tv.fxs = (float)tv.XS;
    tv.fys = (float)tv.YS;
    tv.fxe = (float)(tv.XE < (int32_t)ta.width ? tv.XE : (int32_t)ta.width);
    tv.fye = (float)(tv.YE < (int32_t)ta.height ? tv.YE : (int32_t)ta.height);
    tv.scene = g / ta.n_views;
    if (drawn) {
        const ViewSrc<kBatch> vs{va, vm};
#pragma unroll
        for (int q = 0; q < 12; ++q) tv.M[q] = vs.m(g)[q];
        tv.c = vs.c(g);
        tv.k = (int32_t)vs.k(g);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const float* m = tv.M + 4 * r;
            tv.mg[r] = 0x1p-20f * (fabsf(m[0]) * ta.span[0] + fabsf(m[1]) * ta.span[1] + fabsf(m[2]) * ta.span[2] +
                                   fabsf(m[3]) + fabsf(tv.c) + 1.0f);
        }
    }
    return tv;
}

// Breadth-first walk of the chunk tree by the workgroup's kWaves waves, nodes
// tested one per lane: all nodes of the top level, then the children of those
// that can reach the tile, down to the groups of chunks (level 1), or until a
// level's frontier does not fit kFront. Returns the level lv of the final
// frontier front[*cur] of *curn nodes (lv >= 2 when it stopped early).
template <bool kBatch, int kWaves>
__device__ __forceinline__ uint32_t walk_tree(const uint4* __restrict__ box, const TileArgs& ta, uint64_t F,
                                              const TileView& tv, uint32_t (*front)[kFront], uint32_t* sh_next,
                                              uint32_t* sh_over, uint32_t* cur, uint32_t* curn)
{
    const uint32_t wave = uniform32(threadIdx.x / kWave);
    const int lane = __lane_id();
    uint32_t lv = top_level(F), c = 0;
    if (threadIdx.x == 0) *sh_next = 0;
    __syncthreads();
    const uint32_t n_top = (uint32_t)level_count(F, lv);
    const uint4* top = box + kNodeWords<kBatch> * ta.lv_off[lv];
    for (uint32_t i0 = wave * kWave; i0 < n_top; i0 += kWaves * kWave) {
        const uint32_t i = i0 + (uint32_t)lane;
        const bool ok = i < n_top && box_reaches<kBatch>(top + kNodeWords<kBatch> * (uint64_t)(i < n_top ? i : 0), ta, tv);
        const uint64_t m = __ballot(ok);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(sh_next, (uint32_t)__popcll(m));
        base = uniform32(base);
        if (ok) front[0][base + lanes_below(m)] = i;
    }
    __syncthreads();
    uint32_t n = *sh_next;
    __syncthreads();
    while (lv >= 2 && n > 0) {
        if (threadIdx.x == 0) {
            *sh_next = 0;
            *sh_over = 0;
        }
        __syncthreads();
        const uint64_t n_child = level_count(F, lv - 1);
        for (uint32_t e = wave; e < n; e += kWaves) {
            const uint32_t node = front[c][e];
            const uint64_t m = test_children<kBatch>(box, ta, n_child, lv, node, tv);
            const uint32_t cnt = (uint32_t)__popcll(m);
            uint32_t base = 0;
            if (lane == 0 && cnt) base = atomicAdd(sh_next, cnt);
            base = uniform32(base);
            if ((m >> lane) & 1ull) {
                const uint32_t pos = base + lanes_below(m);
                if (pos < kFront) front[c ^ 1][pos] = node * kFan + (uint32_t)lane;
                else *sh_over = 1;
            }
        }
        __syncthreads();
        const uint32_t nn = *sh_next, over = *sh_over;
        __syncthreads();
        if (over) break;   // keep the current frontier; depth first from here
        c ^= 1;
        n = nn;
        --lv;
    }
    *cur = c;
    *curn = n;
    return n == 0 ? 1 : lv;
}

// Estimate pass, one wave per tile: the walk down to the groups of chunks
// that can reach the tile sets how many workgroups draw it (P, reserved from
// the launch's extra budget: counter 8) and the class of their share of
// groups (0 for nothing to draw, then 1 + log2 of the share, at most 7). Its
// items (tile << 5 | part) go to its class's list, items[class * item_cap +
// rank ...] (counter `class` counts the class's items); parts[tile] = P |
// (1 + listed groups, or 0) << 8, the groups listed in glist[tile *
// kGroupList ...].
//
// A workgroup's 16 tiles add to a class's counter at once, and the counters
// lie in lines of their own: adds on one line run one after the other at the
// memory side, about 9 ns each, and with one per tile they bound the pass
// (30,720 tiles 364 us, here 60).
constexpr uint32_t kEstFront = 128;   // a wave's frontier capacity above the groups

template <bool kBatch>
__global__ void __launch_bounds__(kEstWaves * kWave)
k_tile_est(const uint64_t* __restrict__ n_frag, TileArgs ta, ViewArgs va, const float* __restrict__ vm,
           const uint4* __restrict__ box, uint32_t* __restrict__ items, uint16_t* __restrict__ parts,
           uint32_t* __restrict__ counter, uint32_t* __restrict__ glist)
{
    __shared__ uint32_t front[kEstWaves][2][kEstFront];
    __shared__ uint32_t of_class[kEstWaves], n_items[kEstWaves], first[8];
    const uint32_t wave = uniform32(threadIdx.x / kWave);
    const int lane = __lane_id();
    const uint32_t tile = blockIdx.x * kEstWaves + wave;
    const uint64_t F = frag_total(n_frag, ta.cap_frag);
    const bool drawn = ta.cap_occ > 0 && F > 0 && tile < ta.n_tiles;
    uint32_t P = 0, cls = 0;
    if (tile < ta.n_tiles) {   // wave-uniform
        const TileView tv = tile_view<kBatch>(tile, ta, va, vm, drawn);
        uint32_t groups = 0;   // groups of chunks that can reach the tile (a large value when uncounted)
        bool over = false;
        if (drawn) {
            uint32_t lv = top_level(F), n = (uint32_t)level_count(F, lv), c = 0, kept = 0;
            // nodes i0 + lane of level l (below end): groups counted and the
            // first ones listed, others kept in the frontier
            auto take = [&](uint32_t l, uint64_t i0, uint64_t end, uint32_t* f) {
                const uint64_t i = i0 + (uint32_t)lane;
                const uint64_t m = __ballot(i < end && box_reaches<kBatch>(box + kNodeWords<kBatch> * (ta.lv_off[l] + (i < end ? i : 0)), ta, tv));
                const bool ok = (m >> lane) & 1ull;
                if (l == 1) {
                    const uint32_t at = groups + lanes_below(m);
                    if (ok && at < kGroupList) glist[(size_t)tile * kGroupList + at] = (uint32_t)i;
                    groups += (uint32_t)__popcll(m);
                } else {
                    const uint32_t at = kept + lanes_below(m);
                    if (ok && at < kEstFront) f[at] = (uint32_t)i;
                    kept += (uint32_t)__popcll(m);
                }
            };
            for (uint32_t i0 = 0; i0 < n; i0 += kWave) take(lv, i0, n, front[wave][0]);
            while (lv >= 2) {
                if (kept > kEstFront) {
                    over = true;
                    break;
                }
                // the frontier's entries were written by this wave's lanes
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                n = kept;
                kept = 0;
                --lv;
                const uint64_t end = level_count(F, lv);
                for (uint32_t e = 0; e < n; ++e)
                    take(lv, (uint64_t)uniform32(front[wave][c][e]) * kFan, end, front[wave][c ^ 1]);
                c ^= 1;
            }
        }
        if (over) groups = 1u << 16;
        if (lane == 0) {
            const uint32_t q = (groups + kSplitGroups - 1) / kSplitGroups;
            P = 1;
            while (P < q && P < kMaxParts) P *= 2;
            if (P > 1 && atomicAdd(counter + 8 * kCounterStep, P - 1) + (P - 1) > split_items(ta.n_tiles)) P = 1;
            const uint32_t share = (groups + P - 1) / P;
            cls = share == 0 ? 0u : (share >= 64 ? 7u : 32u - __builtin_clz(share));
            parts[tile] = (uint16_t)(P | ((groups <= kGroupList ? groups + 1 : 0u) << 8));
        }
    }
    if (lane == 0) {
        of_class[wave] = cls;
        n_items[wave] = P;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        uint32_t n = 0;
        for (uint32_t w = 0; w < kEstWaves; ++w) n += of_class[w] == threadIdx.x ? n_items[w] : 0u;
        first[threadIdx.x] = n ? atomicAdd(counter + threadIdx.x * kCounterStep, n) : 0u;
    }
    __syncthreads();
    if (lane == 0 && P > 0) {
        uint32_t r = first[cls];
        for (uint32_t w = 0; w < wave; ++w) r += of_class[w] == cls ? n_items[w] : 0u;
        uint32_t* it = items + (size_t)cls * (ta.n_tiles + split_items(ta.n_tiles)) + r;
        for (uint32_t i = 0; i < P; ++i) it[i] = (tile << 5) | i;
    }
}

// One workgroup per item: a 64 x 64 tile of one view slot, or a sub-tile
// of one (items in the estimate's order; one per tile, in the plain order,
// for launches of 2^22 tiles or more). The chunk tree is walked from its
// top level breadth first (children tested one per lane) down to the groups of
// 64 chunks that can reach the workgroup's sub-tile; then, in rounds of one
// group per wave, the chunks of those groups that can reach it are queued
// in LDS and drawn by all waves in turn into the z-tile in LDS with 64-bit
// minima (fragments outside the sub-tile rejected). Should a level's
// frontier not fit in LDS, every chunk below the last frontier that did is
// drawn. Then each pixel of the sub-tile is written once.
template <int kMode, bool kBatch>
__global__ void __launch_bounds__(kTileThreads, 8)   // 8 waves per SIMD (two workgroups per compute unit): 64 registers
k_tile_splat(const uint4* __restrict__ frag, const uint64_t* __restrict__ pos, const uint64_t* __restrict__ n_frag,
             TileArgs ta, ViewArgs va, const float* __restrict__ vm, const uint4* __restrict__ box,
             const uint16_t* __restrict__ parts, const uint32_t* __restrict__ items,
             const uint32_t* __restrict__ counter, const uint32_t* __restrict__ glist,
             unsigned long long* __restrict__ zbuf, uint32_t* __restrict__ rgba, float* __restrict__ depth,
             uint8_t* __restrict__ cov)
{
    __shared__ unsigned long long zt[kTilePix];
    __shared__ uint32_t front[2][kFront];
    __shared__ uint32_t queue[kTileWaves * kFan];
    __shared__ uint32_t sh_next, sh_over, sh_q;
    uint32_t tile, part = 0, P = 1, listed = 0;
    if (ta.n_tiles < kOrderTiles) {
        // item blockIdx.x of the classes' lists taken from class 7 down
        uint32_t b = blockIdx.x, c = 8;
        for (;;) {
            if (c == 0) return;   // whole workgroup: past the last item
            --c;
            const uint32_t n = counter[c * kCounterStep];
            if (b < n) break;
            b -= n;
        }
        const uint32_t it = items[(size_t)c * (ta.n_tiles + split_items(ta.n_tiles)) + b];
        tile = uniform32(it >> 5);
        part = uniform32(it & 31u);
        const uint32_t pw = uniform32(parts[tile]);
        P = pw & 0xFFu;
        listed = pw >> 8;
    } else {
        tile = uniform32(die_major(blockIdx.x, ta.n_tiles));
    }
    const uint64_t F = frag_total(n_frag, ta.cap_frag);
    const bool drawn = ta.cap_occ > 0 && F > 0;
    const TileView tv = tile_view<kBatch>(tile, ta, va, vm, drawn, part, P);
    for (int p = threadIdx.x; p < kTilePix; p += kTileThreads) zt[p] = ~0ull;
    // the groups the estimate listed for the tile, as the walk's last frontier
    if (listed > 0 && threadIdx.x < listed - 1) front[0][threadIdx.x] = glist[(size_t)tile * kGroupList + threadIdx.x];
    __syncthreads();
    if (drawn) {
        const uint32_t wave = uniform32(threadIdx.x / kWave);
        const int lane = __lane_id();
        uint32_t cur = 0, curn = listed > 0 ? listed - 1 : 0, lv = 1;
        if (listed == 0) lv = walk_tree<kBatch, kTileWaves>(box, ta, F, tv, front, &sh_next, &sh_over, &cur, &curn);
        const uint32_t* fr = front[cur];
        const uint64_t n_chunk = level_count(F, 0);
        if (lv <= 1) {
            // rounds: every wave tests one group's chunks and queues those
            // that can reach the tile (its sub-tile); all waves then
            // draw the queue
            for (uint32_t r0 = 0; r0 < curn; r0 += kTileWaves) {
                if (threadIdx.x == 0) sh_q = 0;
                __syncthreads();
                const uint32_t e = r0 + wave;
                if (e < curn) {
                    const uint32_t node = fr[e];
                    const uint64_t m = test_children<kBatch>(box, ta, n_chunk, 1, node, tv);
                    const uint32_t cnt = (uint32_t)__popcll(m);
                    uint32_t base = 0;
                    if (lane == 0 && cnt) base = atomicAdd(&sh_q, cnt);
                    base = uniform32(base);
                    if ((m >> lane) & 1ull) queue[base + lanes_below(m)] = node * kFan + (uint32_t)lane;
                }
                __syncthreads();
                const uint32_t nq = sh_q;
                draw_queue<kMode, kBatch>(queue, 0, wave, kTileWaves, nq, pos, ta, tv, zt);
                __syncthreads();
            }
        } else {
            // a frontier too large for LDS (a tile that the whole scene
            // projects into): every chunk below each frontier node is drawn,
            // the fragments outside the tile rejected one by one
            for (uint32_t e = 0; e < curn; ++e) {
                uint64_t lo = fr[e];
                for (uint32_t l = 0; l < lv; ++l) lo *= kFan;
                const uint64_t span = lo + ((uint64_t)1 << (6 * lv)) < n_chunk ? (uint64_t)1 << (6 * lv) : n_chunk - lo;
                draw_queue<kMode, kBatch>(nullptr, lo, wave, kTileWaves, (uint32_t)span, pos, ta, tv, zt);
            }
        }
    }
    __syncthreads();
    const uint32_t g = tile / ta.per_view;
    const uint64_t plane = (uint64_t)ta.width * ta.height;
    const uint32_t* f32 = (const uint32_t*)frag;
    for (int p = threadIdx.x; p < kTilePix; p += kTileThreads) {
        const int32_t X = tv.X0 + (p % kTile), Y = tv.Y0 + (p / kTile);
        if (X < tv.XS || X >= tv.XE || Y < tv.YS || Y >= tv.YE || X >= (int32_t)ta.width || Y >= (int32_t)ta.height)
            continue;
        const uint64_t o = (uint64_t)g * plane + (uint64_t)Y * ta.width + (uint32_t)X;
        const unsigned long long zk = zt[p];
        zbuf[o] = zk;
        if (zk == ~0ull) {
            rgba[o] = 0u;
            depth[o] = 0.0f;
            cov[o] = 0;
        } else {
            rgba[o] = f32[4ull * (uint32_t)zk + 1];
            depth[o] = __uint_as_float((uint32_t)(zk >> 32));
            cov[o] = 1;
        }
    }
}

TileArgs tile_args(uint32_t n_scenes, uint32_t n_views, uint32_t W, uint32_t H, uint64_t cap_frag, bool batch)
{
    TileArgs ta{};
    ta.scenes = batch ? 1 : 0;
    ta.n_scenes = n_scenes;
    ta.n_views = n_views;
    ta.width = W;
    ta.height = H;
    ta.nx = (W + kTile - 1) / kTile;
    ta.ny = (H + kTile - 1) / kTile;
    ta.per_view = ta.nx * ta.ny;
    ta.n_tiles = n_scenes * n_views * ta.per_view;
    ta.shift = 64;
    ta.cap_frag = cap_frag;
    ta.levels = top_level(cap_frag) + 1;
    uint64_t off = 0;
    for (uint32_t l = 0; l < ta.levels; ++l) {
        const uint32_t sh = 6 * (l + 1);
        const uint64_t n = (cap_frag + ((uint64_t)1 << sh) - 1) >> sh;
        ta.lv_off[l] = off;
        off += n ? n : 1;
    }
    ta.n_nodes = off;
    return ta;
}

// Span and box units of octant positions of gbits bits.
void octant_units(TileArgs& ta)
{
    ta.qs = ta.gbits > 16 ? ta.gbits - 16 : 0;
    ta.inset = 0.5f;
    for (int k = 0; k < 3; ++k) {
        ta.span[k] = (float)(1u << ta.gbits);
        ta.unit[k] = (float)(1u << ta.qs);
    }
}

// Workspace: the tree's boxes, then the packed positions (a whole number of
// chunks).
size_t tile_pos_off(const TileArgs& ta)
{
    return ((size_t)ta.n_nodes * (ta.scenes ? 2 : 1) * sizeof(uint4) + 255) & ~(size_t)255;
}

// Then, from tile_split_off: 9 counters in lines of their own, and for
// ordered launches the items' lists of the 8 classes (each with room for all
// items), kGroupList group ids per tile and the parts of each tile.
constexpr size_t kCounters = 9 * kCounterStep;

size_t tile_split_off(const TileArgs& ta)
{
    return (tile_pos_off(ta) + (size_t)((ta.cap_frag + kChunk - 1) / kChunk) * kChunk * sizeof(uint64_t) + 255) &
           ~(size_t)255;
}

size_t tile_ws_bytes(const TileArgs& ta)
{
    const size_t cap = ta.n_tiles < kOrderTiles ? (size_t)ta.n_tiles + split_items(ta.n_tiles) : 0;
    const size_t lists = cap ? (size_t)ta.n_tiles * kGroupList : 0;
    return tile_split_off(ta) + (8 * cap + kCounters + lists + (ta.n_tiles + 1) / 2) * sizeof(uint32_t) + 256;
}

template <bool kBatch>
hipError_t tiles_launch(const Device& dev, const fhv_pofa* a, int mode, TileArgs ta, const ViewArgs& va,
                        const float* vm, void* ws, uint64_t* zbuf, uint32_t* rgba, float* depth, uint8_t* cov,
                        hipStream_t s)
{
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    uint4* box = (uint4*)base;
    uint64_t* pos = (uint64_t*)(base + tile_pos_off(ta));
    const bool ordered = ta.n_tiles < kOrderTiles;
    uint32_t* bucket = (uint32_t*)(base + tile_split_off(ta));
    uint32_t* items = bucket + kCounters;   // and the rest: ordered launches only
    uint32_t* glist = items + 8 * ((size_t)ta.n_tiles + split_items(ta.n_tiles));
    uint16_t* parts = (uint16_t*)(glist + (size_t)ta.n_tiles * kGroupList);
    const uint64_t chunks = (a->cap_frag + kChunk - 1) / kChunk;
    const uint64_t gmax = (uint64_t)dev.cus * 16;
    auto grid_for = [&](uint64_t waves) {
        uint64_t gb = (waves + (kBlock / kWave) - 1) / (kBlock / kWave);
        return (unsigned)(gb < 1 ? 1 : (gb > gmax ? gmax : gb));
    };
    hipError_t e;
    {
        ProfScope ps(dev, "splat.bin", s);
        const uint64_t groups = (chunks + kFan - 1) / kFan, gg = (uint64_t)dev.cus * 8;
        const dim3 gb((unsigned)(groups < 1 ? 1 : groups > gg ? gg : groups));
        if (mode == FHV_PPFL)
            k_chunk_box<FHV_PPFL, kBatch><<<gb, dim3(kBoxWaves * kWave), 0, s>>>(
                (const uint4*)a->frag, a->oct_key, a->n_frag, ta, box, pos, bucket);
        else
            k_chunk_box<FHV_POFL, kBatch><<<gb, dim3(kBoxWaves * kWave), 0, s>>>(
                (const uint4*)a->frag, a->oct_key, a->n_frag, ta, box, pos, bucket);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        for (uint32_t l = 2; l < ta.levels; ++l) {
            const uint64_t nodes = (l + 1 < ta.levels ? ta.lv_off[l + 1] : ta.n_nodes) - ta.lv_off[l];
            k_node_box<kBatch><<<dim3(grid_for(nodes)), dim3(kBlock), 0, s>>>(a->n_frag, ta, l, box);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    if (ordered) {
        ProfScope ps(dev, "splat.est", s);
        k_tile_est<kBatch><<<dim3((ta.n_tiles + kEstWaves - 1) / kEstWaves), dim3(kEstWaves * kWave), 0, s>>>(a->n_frag, ta, va, vm, box, items,
                                                                                  parts, bucket, glist);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    ProfScope ps(dev, "splat.splat", s);
    const dim3 grid(ta.n_tiles + split_items(ta.n_tiles));
    if (mode == FHV_PPFL)
        k_tile_splat<FHV_PPFL, kBatch><<<grid, dim3(kTileThreads), 0, s>>>(
            (const uint4*)a->frag, pos, a->n_frag, ta, va, vm, box, parts, items, bucket, glist,
            (unsigned long long*)zbuf, rgba, depth, cov);
    else
        k_tile_splat<FHV_POFL, kBatch><<<grid, dim3(kTileThreads), 0, s>>>(
            (const uint4*)a->frag, pos, a->n_frag, ta, va, vm, box, parts, items, bucket, glist,
            (unsigned long long*)zbuf, rgba, depth, cov);
    return hipGetLastError();
}

}  // namespace

bool splat_fits(uint64_t cap_frag, uint32_t n_scenes, uint32_t n_views, uint32_t width, uint32_t height)
{
    const uint64_t tiles = (uint64_t)n_scenes * n_views * ((width + kTile - 1) / kTile) * ((height + kTile - 1) / kTile);
    return tiles < (1ull << 31) && (cap_frag + kChunk - 1) / kChunk < (1ull << 32);
}

size_t splat_ws_bytes(uint64_t cap_frag, uint32_t n_scenes, uint32_t n_views, uint32_t width, uint32_t height,
                      bool batch)
{
    return tile_ws_bytes(tile_args(n_scenes, n_views, width, height, cap_frag, batch));
}

hipError_t splat_launch(const Device& dev, const fhv_pofa* a, const fhv_capture_desc* d, const ViewArgs& va,
                        uint64_t* zbuf, uint32_t* rgba, float* depth, uint8_t* cov, void* ws, hipStream_t s)
{
    TileArgs ta = tile_args(1, va.n_views, va.width, va.height, a->cap_frag, false);
    ta.cap_w = d->width;
    ta.cap_occ = a->cap_occ;
    ta.gbits = d->levels + 8;
    if (d->mode == FHV_PPFL) {
        ta.span[0] = (float)d->width;
        ta.span[1] = (float)d->height;
        ta.span[2] = 16777216.0f;
        ta.unit[0] = ta.unit[1] = 1.0f;
        ta.unit[2] = 256.0f;
        ta.inset = 0.0f;   // depths are taken as they are
    } else {
        octant_units(ta);
    }
    return tiles_launch<false>(dev, a, (int)d->mode, ta, va, nullptr, ws, zbuf, rgba, depth, cov, s);
}

hipError_t splat_batch_launch(const Device& dev, const fhv_pofa* a, uint32_t levels, const BatchViews& bv,
                              uint64_t* zbuf, uint32_t* rgba, float* depth, uint8_t* cov, void* ws, hipStream_t s)
{
    TileArgs ta = tile_args(bv.n_scenes, bv.n_views, bv.width, bv.height, a->cap_frag, true);
    ta.shift = 3 * levels;
    ta.cap_occ = a->cap_occ;
    ta.gbits = levels + 8;
    octant_units(ta);
    ViewArgs va;
    memset(&va, 0, sizeof(va));
    va.n_views = bv.n_views;
    va.width = bv.width;
    va.height = bv.height;
    va.k[0] = bv.k;
    va.c[0] = 0.5f - 0.5f * (float)bv.k;
    return tiles_launch<true>(dev, a, FHV_POFL, ta, va, bv.m, ws, zbuf, rgba, depth, cov, s);
}

}  // namespace fhv
