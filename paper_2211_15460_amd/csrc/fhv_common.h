// Device-side definitions shared by the HIP translation units of libfhv.
// gfx950 (CDNA4) only: wave64, 64-bit atomics on global memory.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/fhv.h"

namespace fhv {

constexpr uint32_t kNil = 0xFFFFFFFFu;
constexpr int kBlock = 256;          // threads per workgroup (4 waves)
constexpr int kWave = 64;
constexpr int kBrickShift = 9;       // compaction bucket: 512 consecutive keys
constexpr uint32_t kBrickKeys = 1u << kBrickShift;
constexpr uint32_t kMaxViews = 32;

// Triangle after setup, oriented counter-clockwise in 16.8 fixed point: its
// sample bounding box and what the rasterizer evaluates at the samples. 256
// bytes, read through the scalar cache; the first 64 hold all that coverage
// needs of a narrow triangle.
//
// A triangle whose box spans W x H fixed-point units with W H <= 2^30 (and
// W, H < 2^22) is narrow: its edge functions at the samples of its box fit 32
// bits, and every interpolated attribute's numerator fits a double, so the
// record holds both as linear forms. Any other triangle is wide: it keeps
// its vertices and takes 64-bit integers.
constexpr uint32_t kTriNarrow = 1u;
constexpr uint32_t kTriDepth32 = 2u;   // narrow PPFL triangle, twice its area >= 2^26

struct TriHead {
    int32_t lo_i, lo_j;       // first sample column / row
    int32_t hi_i, hi_j;       // last sample column / row (inclusive)
    uint32_t tiles_x;         // tiles per bbox row
    uint32_t flags;           // kTri*
    uint32_t nrm;             // packed normal
    uint32_t aux;             // object byte << 24
    // narrow: edge functions 01, 12 and 20 at sample (lo_i, lo_j), each less
    // one unless the edge owns its samples (top-left rule): a sample is
    // covered when none of the three is negative. Edges 01 and 12 change by
    // 256 ex per sample column and 256 ey per row, edge 20 by minus their sum.
    int32_t e0[3], ex[2], ey[2];
    uint32_t scene;           // scene of a batch (key space offset scene << 3L)
};

// Attribute at a covered sample of a narrow triangle: floor of
// (d0 e12 + d1 e20 + c) / A, e12 and e20 as in the head.
struct TriAtt {
    double d0, d1, c;
};

struct TriNarrow {
    TriAtt att[7];            // R, G, B, A, then grid x, y, z (POFL) or depth24 (PPFL)
};

// kTriDepth32: the depth's numerator may exceed 2^53; it is then an estimate,
// corrected by the remainder modulo 2^32 from the vertices' depths, twice the
// area and the rounding term. At the end of the PPFL records' attributes.
struct TriDepth {
    uint32_t z[3], A, half, pad;
};

struct TriWide {
    int32_t x[3], y[3];       // 16.8 screen (PPFL) or tangent plane (POFL)
    uint32_t rgba[3];
    int32_t a[3][3];          // PPFL: a[k][0] = depth24; POFL: grid xyz
    int64_t A;                // twice the area, > 0
};

struct alignas(64) TriRec {
    TriHead h;
    double rA;                // 1 / A
    union {
        TriNarrow n;
        struct {
            TriAtt skip[5];
            TriDepth d;
        };
        TriWide w;
    };
    uint32_t pad[4];
};
static_assert(sizeof(TriHead) == 64 && sizeof(TriRec) == 256, "TriRec layout");

struct ViewArgs {
    float m[kMaxViews][12];
    float c[kMaxViews];       // 1/2 - k/2
    uint32_t k[kMaxViews];
    uint32_t n_views;
    uint32_t width;
    uint32_t height;
    uint32_t all_k1;        // every view has a one-pixel footprint
};

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t uniform32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

__device__ __forceinline__ uint64_t lanemask_lt()
{
    return (1ull << __lane_id()) - 1ull;
}

// The active lanes of the wave whose value equals this lane's, as a bit mask
// (0 for an inactive lane): one pass per distinct value, no memory involved.
// Must be called by all lanes of the wave.
__device__ __forceinline__ uint64_t wave_same(uint32_t v, bool active)
{
    uint64_t todo = __ballot(active), mine = 0;
    while (todo) {
        const uint32_t lv = (uint32_t)__builtin_amdgcn_readlane((int)v, __builtin_ctzll(todo));
        const uint64_t m = __ballot(v == lv) & todo;
        if (active && v == lv) mine = m;
        todo &= ~m;
    }
    return mine;
}

// Inclusive sum and maximum over the wave in registers (data-parallel
// primitives: shifts within rows of 16 lanes, then across the rows).
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15 to rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31 to rows 2, 3
    return v;
}

__device__ __forceinline__ uint32_t wave_all_max(uint32_t v)
{
    auto m = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = m(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xF, 0xF, false));   // row_ror:8
    v = m(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x124, 0xF, 0xF, false));
    v = m(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x122, 0xF, 0xF, false));
    v = m(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x121, 0xF, 0xF, false));
    return m(m((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
             m((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Spread the low 21 bits of v to every third bit (bit b -> bit 3b).
__device__ __forceinline__ uint64_t spread3(uint32_t v32)
{
    uint64_t v = v32 & 0x1FFFFFull;
    v = (v | (v << 32)) & 0x1F00000000FFFFull;
    v = (v | (v << 16)) & 0x1F0000FF0000FFull;
    v = (v | (v << 8)) & 0x100F00F00F00F00Full;
    v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// spread3 of a 10-bit value in 32 bits.
__device__ __forceinline__ uint32_t spread3_10(uint32_t v)
{
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

// Inverse of spread3_10.
__device__ __forceinline__ uint32_t compact3_10(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    return (v | (v >> 16)) & 0x3FFu;
}

// Inverse of spread3: every third bit of v (bit 3b -> bit b).
__device__ __forceinline__ uint32_t compact3(uint64_t v)
{
    v &= 0x1249249249249249ull;
    v = (v | (v >> 2)) & 0x10C30C30C30C30C3ull;
    v = (v | (v >> 4)) & 0x100F00F00F00F00Full;
    v = (v | (v >> 8)) & 0x1F0000FF0000FFull;
    v = (v | (v >> 16)) & 0x1F00000000FFFFull;
    v = (v | (v >> 32)) & 0x1FFFFFull;
    return (uint32_t)v;
}

// Bounding box of integer positions over a run of fragments: per axis the
// lowest and highest value in units that fit 16 bits; empty where lo > hi.
// Kept as minima of (lo, 65535 - hi) while it is built: three words of two
// values. As stored (box_store): lo x | lo y << 16, lo z | hi x << 16,
// hi y | hi z << 16.
struct BoxMin {
    uint32_t v[3];
};

__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t,
                              __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Minimum over the wave, in registers: rotations within rows of 16 lanes,
// then the four rows.
__device__ __forceinline__ uint32_t wave_pk_min(uint32_t v)
{
    v = pk_min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xF, 0xF, false));   // row_ror:8
    v = pk_min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x124, 0xF, 0xF, false));
    v = pk_min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x122, 0xF, 0xF, false));
    v = pk_min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x121, 0xF, 0xF, false));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16),
                   c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return pk_min(pk_min(a, b), pk_min(c, d));
}

__device__ __forceinline__ BoxMin box_join(const BoxMin& a, const BoxMin& b)
{
    return BoxMin{{pk_min(a.v[0], b.v[0]), pk_min(a.v[1], b.v[1]), pk_min(a.v[2], b.v[2])}};
}

// The box of the wave's positions (in its units), of the lanes with ok.
__device__ __forceinline__ BoxMin wave_box(uint32_t x, uint32_t y, uint32_t z, bool ok)
{
    return BoxMin{{wave_pk_min(ok ? x | (y << 16) : ~0u), wave_pk_min(ok ? z | ((0xFFFFu - x) << 16) : ~0u),
                   wave_pk_min(ok ? (0xFFFFu - y) | ((0xFFFFu - z) << 16) : ~0u)}};
}

__device__ __forceinline__ uint4 box_store(const BoxMin& m)
{
    return make_uint4(m.v[0], m.v[1] ^ 0xFFFF0000u, ~m.v[2], 0u);
}

__device__ __forceinline__ BoxMin box_load(const uint4& b)
{
    return BoxMin{{b.x, b.y ^ 0xFFFF0000u, ~b.z}};
}

}  // namespace fhv

// Launchers (host side), defined next to their kernels.
namespace fhv {

struct Profiler;  // kernel timing with HIP events, owned by the context

// Launch choices (fhv_tuning): raster tile width (8, 16 or 32 samples; a
// tile is 64 samples), workgroups per compute unit of the rasterizer; the
// last one is kept for its caller and reaches no launch.
struct Tuning {
    uint32_t tile_w = 8;
    uint32_t raster_wg = 16;
    uint32_t splat_wg = 16;
};

struct Device {
    int id;
    int cus;
    Profiler* prof;  // non-null while profiling is on
    Tuning tune;
};

void prof_mark(Profiler* p, const char* name, hipStream_t s, bool start);

// Brackets the kernel launches of one scope with events when profiling.
struct ProfScope {
    Profiler* p;
    const char* name;
    hipStream_t s;
    ProfScope(const Device& d, const char* n, hipStream_t st) : p(d.prof), name(n), s(st)
    {
        if (p) prof_mark(p, name, s, true);
    }
    ~ProfScope()
    {
        if (p) prof_mark(p, name, s, false);
    }
};

// zero: a counter to clear in the same launch, or null
hipError_t fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s, uint64_t* zero = nullptr);
hipError_t fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s);

// Exclusive (or inclusive) prefix sums of n values; `partial` needs
// scan_partials(n) elements; *total (device, may be null) gets the sum.
size_t scan_partials(uint64_t n);
hipError_t scan_u32(const uint32_t* in, uint32_t* out, uint64_t n, bool inclusive,
                    uint32_t* partial, uint64_t* total, hipStream_t s);
hipError_t scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, bool inclusive,
                    uint64_t* partial, uint64_t* total, hipStream_t s);

// Scenes of a batch: triangle t belongs to the scene s with
// scene_tri[s] <= t < scene_tri[s + 1]; its keys are offset by s << 3L.
struct Scenes {
    const uint32_t* scene_tri;
    uint32_t n_scenes;
};

size_t capture_ws_bytes(const fhv_capture_desc* d, uint32_t n_tri);
hipError_t capture_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d,
                          const fhv_lists* L, void* ws, hipStream_t s, const Scenes* sc = nullptr);

size_t compact_ws_bytes(const fhv_capture_desc* d, uint64_t n_head, uint64_t capacity);
hipError_t compact_launch(const Device& dev, const fhv_lists* L, const fhv_capture_desc* d,
                          const fhv_pofa* out, void* ws, hipStream_t s);

// Splat workspace for arrays of cap_frag records into n_scenes x n_views
// views of width x height (batch: boxes with scene ranges).
size_t splat_ws_bytes(uint64_t cap_frag, uint32_t n_scenes, uint32_t n_views, uint32_t width, uint32_t height,
                      bool batch = false);
// Whether the splat's bins of such a call fit its 32-bit offsets.
bool splat_fits(uint64_t cap_frag, uint32_t n_scenes, uint32_t n_views, uint32_t width, uint32_t height);
hipError_t splat_launch(const Device& dev, const fhv_pofa* a, const fhv_capture_desc* d,
                        const ViewArgs& va, uint64_t* zbuf, uint32_t* rgba, float* depth,
                        uint8_t* cov, void* ws, hipStream_t s);

// Views of a batch: matrices [n_scenes][n_views][12] in device memory.
struct BatchViews {
    const float* m;
    uint32_t n_scenes, n_views, width, height, k;
};

hipError_t splat_batch_launch(const Device& dev, const fhv_pofa* a, uint32_t levels, const BatchViews& bv,
                              uint64_t* zbuf, uint32_t* rgba, float* depth, uint8_t* cov, void* ws,
                              hipStream_t s);

// Two-pass capture straight into per-octant arrays (fhv_capture_arrays):
// the rasterizer counts fragments per brick (kActCount) or stores each at its
// brick's next free staging slot (kActInsert) instead of appending to lists.
enum RasterAct { kActList = 0, kActCount = 1, kActInsert = 2 };
// Passes of fewer tiles than this have fewer than 2^30 fragments, so that the
// 32-bit sums of all three passes over the axes hold them.
constexpr uint64_t kManyTiles = 1ull << 24;
struct BrickSink {
    uint32_t* cnt;                  // kActCount: per-brick counts
    const uint32_t* off;            // kActInsert: brick offsets in the staging array
    uint32_t* cur;                  //             per-brick slot cursors (zeroed)
    uint4* stage;                   //             staging records, w3 = key within the brick
    const uint32_t* skip;           //             non-zero: the arrays are too small, store nothing
    unsigned long long* total;      // kActCount: fragments of passes of kManyTiles tiles or more (zeroed)
};
// again: the records of the call before (same mesh and workspace) are still
// there, so a single-pass projection need not set them up anew.
hipError_t capture_bricks_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d, void* ws,
                                 int act, const BrickSink& bs, bool again, hipStream_t s);
size_t capture_arrays_ws_bytes(const fhv_capture_desc* d, uint32_t n_tri, uint64_t capacity);
hipError_t capture_arrays_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d,
                                 const fhv_pofa* out, void* ws, hipStream_t s);

// Shading of splat winners (fhv_shade): per view the light, viewer and half
// vectors and the material terms.
struct ShadeArgs {
    float l[kMaxViews][3], v[kMaxViews][3], h[kMaxViews][3];
    float ka[kMaxViews], kd[kMaxViews], ks[kMaxViews];
    uint32_t shine[kMaxViews];
};
hipError_t shade_launch(const Device& dev, const fhv_pofa* p, const uint64_t* zbuf, uint32_t n_views,
                        uint64_t n_pix, const ShadeArgs& a, float* out, hipStream_t s);

// Ray casting of per-octant arrays (fhv_raycast): octree depth up to
// kMaxRayLevels (Morton codes of octants fit 32 bits).
constexpr uint32_t kMaxRayLevels = 10;
struct RayViews {
    float m[kMaxViews][12];
    uint32_t n_views, width, height;
};
size_t raycast_ws_bytes(uint32_t levels);
hipError_t raycast_launch(const Device& dev, const fhv_pofa* p, uint32_t levels, const RayViews& rv,
                          uint32_t mode, float tau, float* out, void* ws, size_t ws_bytes, hipStream_t s);

// Measurement probes (fhv_probe): copy over the buffer's two halves, or
// one atomic per line and pass.
hipError_t probe_launch(const Device& dev, uint32_t kind, void* buf, uint64_t bytes, uint32_t line,
                        uint32_t passes, hipStream_t s);

namespace nn {
uint64_t param_count(uint32_t levels);
size_t fill_ws_bytes(uint32_t levels, uint32_t N, uint32_t H, uint32_t W, bool training, bool trace = false);
uint32_t trace_tensors(uint32_t levels, uint32_t N, uint32_t H, uint32_t W, fhv_fill_tensor* out, uint32_t cap);
hipError_t fill(const Device& dev, uint32_t levels, const float* th, const uint32_t* rgba, const float* depth,
                const uint8_t* cov, uint32_t N, uint32_t H, uint32_t W, uint32_t* out, float* residual,
                void* ws, hipStream_t s);
hipError_t train_step(const Device& dev, uint32_t levels, float* th, float* m, float* v, uint32_t step,
                      float lr, const uint32_t* rgba, const float* depth, const uint8_t* cov,
                      const uint32_t* tgt, uint32_t N, uint32_t H, uint32_t W, float* loss, float* grad_out,
                      void* ws, hipStream_t s, bool trace);
}  // namespace nn

// Workspace carving with 256-byte alignment.
struct Carver {
    char* base;
    size_t off;
    template <class T>
    T* take(uint64_t n)
    {
        off = (off + 255) & ~(size_t)255;
        T* p = base ? (T*)(base + off) : nullptr;
        off += (size_t)n * sizeof(T);
        return p;
    }
};

}  // namespace fhv
