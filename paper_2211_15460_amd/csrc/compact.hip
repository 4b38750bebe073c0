// Compaction of fragment lists into per-octant arrays (FHV_POFA, Sec. 3.1
// Fig. 6 and Sec. 3.2): per occupied key a count and an offset, the offsets
// being sums of counts in ascending key (Morton) order, every key's records
// contiguous, ascending by (w0, w1, w2), w3 = the key's table rank.
//
// The paper counts per octant, scans, resets the counters and rasterizes a
// second time. Here the pool's keys are read linearly instead, from the
// sidecar the capture wrote, and keys are grouped in buckets ("bricks") of
// 512 consecutive keys so that every bucket fits a workgroup's LDS:
//   k_hist     per brick: fragment count; every pool slot's place among its
//              brick's fragments
//   scan       exclusive sums of the brick counts: brick fragment offsets
//              and the list of occupied bricks; total = n_frag
//   k_scatter  every pool index to its place in its brick's range, with the
//              key's low 9 bits (the key inside the brick)
//   k_brick_occ  per occupied brick: distinct keys
//   scan       exclusive sums of the distinct-key counts over the list:
//              brick rank bases; total = n_occ
//   k_bricks / k_bricks_large
//              per brick: its records gathered from the pool, counting sort
//              by key inside LDS, each record's rank inside its key's run in
//              canonical order, then the output records with w3 = rank and
//              the brick's table rows. Bricks of up to 256 records take one
//              wave each with no workgroup barriers, up to 1024 a workgroup
//              of 4 waves; the second kernel takes larger ones (in LDS up to
//              8192 records, in memory beyond)
//
// Bytes per fragment (32-bit keys): key 4 read twice, place 4 written and
// read, index and low key 8 written and read twice, record 16 read, 16
// written, and 16 per occupied octant.
#include <algorithm>

#include "scan.h"

namespace fhv {

namespace {

__device__ __forceinline__ uint64_t frag_count(const uint64_t* counter, uint64_t cap)
{
    const uint64_t c = *counter;
    return c < cap ? c : cap;
}

// An occupied brick, in the list that the count scan writes: brick, offset
// of its first fragment, fragments; z in .w: distinct keys, then (after the
// second scan) the rank of its first key.
typedef uint4 BrickEntry;

// Brick counts, and each slot's place in its brick. The lanes of a wave with
// the same brick are found in registers; their leader adds them to the
// workgroup's own counter of the brick in LDS, and one memory atomic per
// brick and workgroup of 2048 slots places the whole workgroup's share: one
// round trip, where an atomic per wave and brick each waited for its own
// result, and few adds where a few bricks take everything (128 x 128 pixel
// keys make 32 bricks). A brick whose LDS counter is taken by another one
// (same low 9 bits) goes to memory directly.
// Hist and scatter of 5.2 M fragments took 69 + 62 us with an atomic per
// wave and brick, and with the distinct keys' bitmap set by atomics here.
constexpr int kHistPer = 8;
constexpr uint32_t kHistSlots = 512;

template <class KeyT>
__global__ void __launch_bounds__(kBlock)
k_hist(const KeyT* __restrict__ keys, const uint64_t* __restrict__ counter, uint64_t cap,
       uint32_t* __restrict__ brick_cnt, uint32_t* __restrict__ place, uint64_t* __restrict__ n_frag)
{
    __shared__ uint32_t tag[kHistSlots], cnt[kHistSlots];
    const uint64_t F = frag_count(counter, cap);
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_frag = F;
    constexpr uint64_t kPer = (uint64_t)kBlock * kHistPer;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kPer; i0 < F; i0 += (uint64_t)gridDim.x * kPer) {
        uint32_t b[kHistPer];
#pragma unroll
        for (int k = 0; k < kHistPer; ++k) {
            const uint64_t i = i0 + (uint64_t)k * kBlock + threadIdx.x;
            b[k] = i < F ? (uint32_t)((uint64_t)keys[i] >> kBrickShift) : kNil;
        }
        for (uint32_t t = threadIdx.x; t < kHistSlots; t += kBlock) {
            tag[t] = kNil;
            cnt[t] = 0;
        }
        __syncthreads();
        uint32_t at[kHistPer];   // LDS slot << 16 | place in the workgroup's share; kNil: place in `far`
        uint32_t far[kHistPer];
#pragma unroll
        for (int k = 0; k < kHistPer; ++k) {
            const bool act = b[k] != kNil;
            const uint64_t same = wave_same(b[k], act);
            const uint32_t rank = lanes_below(same);
            uint32_t v = 0, f = 0;
            if (act && rank == 0) {
                const uint32_t h = b[k] & (kHistSlots - 1), n = (uint32_t)__popcll(same);
                const uint32_t old = atomicCAS(tag + h, kNil, b[k]);
                if (old == kNil || old == b[k]) {
                    v = (h << 16) | atomicAdd(cnt + h, n);
                } else {
                    v = kNil;
                    f = atomicAdd(brick_cnt + b[k], n);
                }
            }
            const int leader = __builtin_ctzll(same | (1ull << 63));
            v = (uint32_t)__shfl((int)v, leader, kWave);
            at[k] = v == kNil ? kNil : v + rank;
            far[k] = 0;
            if (__ballot(act && v == kNil)) far[k] = (uint32_t)__shfl((int)f, leader, kWave) + rank;
        }
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < kHistSlots; t += kBlock)
            if (cnt[t]) cnt[t] = atomicAdd(brick_cnt + tag[t], cnt[t]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kHistPer; ++k) {
            const uint64_t i = i0 + (uint64_t)k * kBlock + threadIdx.x;
            if (i < F) place[i] = at[k] == kNil ? far[k] : cnt[at[k] >> 16] + (at[k] & 0xFFFFu);
        }
        __syncthreads();
    }
}

template <class KeyT>
__global__ void __launch_bounds__(kBlock)
k_scatter(const KeyT* __restrict__ keys, const uint64_t* __restrict__ counter, uint64_t cap,
          const uint32_t* __restrict__ brick_off, const uint32_t* __restrict__ place, uint2* __restrict__ ent)
{
    const uint64_t F = frag_count(counter, cap);
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    constexpr int kU = 4;   // slots in flight per thread
    for (uint64_t i0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i0 < F; i0 += kU * stride) {
        uint64_t key[kU];
        uint32_t p[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t i = i0 + u * stride;
            key[u] = i < F ? (uint64_t)keys[i] : 0;
            p[u] = i < F ? place[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) p[u] += brick_off[key[u] >> kBrickShift];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t i = i0 + u * stride;
            if (i < F) ent[p[u]] = make_uint2((uint32_t)i, (uint32_t)key[u] & (kBrickKeys - 1));
        }
    }
}

// Outputs that overlap the pool (arrays made in place of the lists): records
// must leave the pool before the sorts write, so every one is copied to its
// brick's range of the staging array, its low key in w3. The staging array
// covers the places of k_hist; slots come from cursors instead, one atomic
// per wave and brick.
template <class KeyT>
__global__ void __launch_bounds__(kBlock)
k_stage(const uint4* __restrict__ pool, const KeyT* __restrict__ keys, const uint64_t* __restrict__ counter,
        uint64_t cap, const uint32_t* __restrict__ brick_off, uint32_t* __restrict__ brick_cur,
        uint4* __restrict__ stage)
{
    const uint64_t F = frag_count(counter, cap);
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    const uint64_t Fw = (F + kWave - 1) & ~(uint64_t)(kWave - 1);   // whole waves take part in wave_same
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < Fw; i += stride) {
        const bool act = i < F;
        const uint64_t key = act ? (uint64_t)keys[i] : 0u;
        const uint32_t b = (uint32_t)(key >> kBrickShift);
        const uint64_t same = wave_same(b, act);
        const uint32_t rank = lanes_below(same);
        uint32_t slot = act && rank == 0 ? atomicAdd(brick_cur + b, (uint32_t)__popcll(same)) : 0u;
        slot = (uint32_t)__shfl((int)slot, __builtin_ctzll(same | (1ull << 63)), kWave) + rank;
        if (!act) continue;
        uint4 r = pool[i];
        r.w = (uint32_t)key & (kBrickKeys - 1);
        stage[brick_off[b] + slot] = r;
    }
}

// Where a brick's records come from: gathered from the pool through the
// scattered indices, or staged whole with the low key in w3 (two-pass
// capture into arrays, arrays made in place of the lists).
template <bool kGather>
struct BrickSrc {
    const uint4* pool;
    uint2* ent;
    uint4* stage;
    __device__ __forceinline__ uint32_t low(uint64_t i) const { return kGather ? ent[i].y : stage[i].w; }
    __device__ __forceinline__ uint4 rec(uint64_t i) const   // w = low key
    {
        if (!kGather) return stage[i];
        const uint2 e = ent[i];
        uint4 r = pool[e.x];
        r.w = e.y;
        return r;
    }
};

// Orders LDS traffic of one wave: its earlier LDS writes are complete and
// visible to all its lanes before later LDS reads.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Distinct keys of every occupied brick, one wave per brick: a bit per key
// in LDS.
template <bool kGather>
__global__ void __launch_bounds__(kBlock)
k_brick_occ(BrickEntry* __restrict__ list, const uint64_t* __restrict__ list_total, BrickSrc<kGather> src)
{
    constexpr int kWords = kBrickKeys / 32;
    __shared__ uint32_t bits[kBlock / kWave][kWords];
    const int lane = __lane_id(), wv = threadIdx.x / kWave;
    const uint32_t nl = (uint32_t)(*list_total >> 32);
    for (uint32_t li = blockIdx.x * (kBlock / kWave) + wv; li < nl; li += gridDim.x * (kBlock / kWave)) {
        const BrickEntry e = list[li];
        if (lane < kWords) bits[wv][lane] = 0;
        wave_lds_sync();
        auto key = [&](uint32_t i) -> uint32_t { return src.low((uint64_t)e.y + i) & (kBrickKeys - 1); };
        uint32_t i = lane;
        for (; i - lane + 4 * kWave <= e.z; i += 4 * kWave) {   // four loads in flight
            uint32_t k[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) k[u] = key(i + u * kWave);
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) atomicOr(&bits[wv][k[u] >> 5], 1u << (k[u] & 31));
        }
        for (; i < e.z; i += kWave) {
            const uint32_t k = key(i);
            atomicOr(&bits[wv][k >> 5], 1u << (k & 31));
        }
        wave_lds_sync();
        uint32_t c = lane < kWords ? (uint32_t)__popc(bits[wv][lane]) : 0u;
#pragma unroll
        for (int d = 1; d < kWords; d <<= 1) c += (uint32_t)__shfl_xor((int)c, d, kWave);
        if (lane == 0) list[li].w = c;
        wave_lds_sync();
    }
}

struct BrickOut {
    uint4* frag;
    uint64_t* oct_key;
    uint32_t *oct_off, *oct_cnt;
    uint64_t cap_occ;
    __device__ __forceinline__ void row(uint64_t rank, uint32_t brick, uint32_t leaf, uint32_t off, uint32_t cnt) const
    {
        if (rank >= cap_occ) return;
        oct_key[rank] = ((uint64_t)brick << kBrickShift) | leaf;
        oct_off[rank] = off;
        oct_cnt[rank] = cnt;
    }
};

// (w0, w1, w2) order; records equal in all three by position p, q.
__device__ __forceinline__ bool rec_before(const uint4& a, uint32_t p, const uint4& b, uint32_t q)
{
    const uint64_t a01 = ((uint64_t)a.x << 32) | a.y, b01 = ((uint64_t)b.x << 32) | b.y;
    return a01 < b01 || (a01 == b01 && (a.z < b.z || (a.z == b.z && p < q)));
}

// Inclusive sums over a group of kT threads (kT = kWave, or a workgroup with
// one total per wave in `tot`).
template <int kT, class T>
__device__ __forceinline__ T group_incl_scan(T v, T* tot)
{
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const T u = __shfl_up(v, d, kWave);
        if (lane >= d) v += u;
    }
    if (kT > kWave) {
        const int wv = threadIdx.x / kWave;
        if (lane == kWave - 1) tot[wv] = v;
        __syncthreads();
        T before = 0;
#pragma unroll
        for (int w = 0; w < kT / kWave; ++w) before += w < wv ? tot[w] : T(0);
        v += before;
    }
    return v;
}

template <int kT>
__device__ __forceinline__ void group_sync()
{
    if (kT == kWave)
        wave_lds_sync();
    else
        __syncthreads();
}

// One brick of n <= kT kPer records by a group of kT threads (thread t of
// it), in LDS: buf holds the records grouped by key, tab[k] the start of
// key k's run | the key's rank in the brick << 16 (tab[kBrickKeys] the end).
// Each record then counts the records of its run that precede it and is
// written straight to its final place. The loads, LDS atomics and the scan
// are chains of latencies: a brick is given as many threads as four records
// each make, and as little LDS as sixteen bytes a record and four a key, so
// that several hide each other.
template <int kT, int kPer, bool kGather>
__device__ __forceinline__ void brick_in_lds(uint32_t t, const BrickEntry& e, const BrickSrc<kGather>& src,
                                             uint4* __restrict__ buf, uint32_t* __restrict__ tab, uint32_t* tot,
                                             const BrickOut& out)
{
    const uint32_t n = e.z, o = e.y, base_rank = e.w;
    uint4 r[kPer];
    uint32_t seq[kPer];   // arrival in the key's run
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t i = t + (uint32_t)(k * kT);
        r[k] = i < n ? src.rec((uint64_t)o + i) : make_uint4(0, 0, 0, 0);
    }
    for (uint32_t k = t; k < kBrickKeys; k += kT) tab[k] = 0;
    group_sync<kT>();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        r[k].w &= kBrickKeys - 1;
        seq[k] = t + (uint32_t)(k * kT) < n ? atomicAdd(tab + r[k].w, 1u) : 0u;
    }
    group_sync<kT>();
    // runs and ranks: kLeaf consecutive keys per thread
    constexpr int kLeaf = kT >= (int)kBrickKeys ? 1 : (int)kBrickKeys / kT;
    uint32_t c[kLeaf], s = 0;
    const bool mine = t * kLeaf < kBrickKeys;
#pragma unroll
    for (int k = 0; k < kLeaf; ++k) {
        c[k] = mine ? tab[t * kLeaf + k] : 0u;
        s += c[k] + (c[k] ? 0x10000u : 0u);
    }
    uint32_t p = group_incl_scan<kT>(s, tot) - s;
    if (mine) {
#pragma unroll
        for (int k = 0; k < kLeaf; ++k) {
            const uint32_t leaf = t * kLeaf + k;
            tab[leaf] = p;
            if (c[k]) out.row((uint64_t)base_rank + (p >> 16), e.x, leaf, o + (p & 0xFFFFu), c[k]);
            p += c[k] + (c[k] ? 0x10000u : 0u);
        }
        if ((t + 1) * kLeaf == kBrickKeys) tab[kBrickKeys] = p;
    }
    group_sync<kT>();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (t + (uint32_t)(k * kT) < n) buf[(tab[r[k].w] & 0xFFFFu) + seq[k]] = r[k];
    group_sync<kT>();
    for (uint32_t q = t; q < n; q += kT) {
        const uint4 x = buf[q];
        const uint32_t lo_rank = tab[x.w], lo = lo_rank & 0xFFFFu, hi = tab[x.w + 1] & 0xFFFFu;
        uint32_t before = 0;
        for (uint32_t d = lo; d < hi; d += 4) {   // four reads in flight
            uint4 y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) y[u] = buf[d + u < hi ? d + u : lo];
#pragma unroll
            for (int u = 0; u < 4; ++u) before += d + u < hi && rec_before(y[u], d + u, x, q) ? 1u : 0u;
        }
        out.frag[(uint64_t)o + lo + before] = make_uint4(x.x, x.y, x.z, base_rank + (lo_rank >> 16));
    }
}

constexpr uint32_t kWaveRecs = 256;     // a wave's brick
constexpr uint32_t kGroupRecs = 1024;   // a 4-wave workgroup's brick
constexpr uint32_t kLdsRecs = 8192;     // a 16-wave workgroup's brick
constexpr uint32_t kTab = kBrickKeys + 1;

// Bricks of up to kGroupRecs records: a workgroup takes four entries of the
// list; each wave sorts its own if it has at most kWaveRecs records, then
// the workgroup the larger ones one after the other. (A launch per size,
// each walking the whole list, with 16 records per lane of one wave for the
// larger bricks and 22 KB of LDS for each, so that seven waves shared a
// compute unit, took 46 + 101 us for 5.2 M fragments in place of this
// kernel.)
template <bool kGather>
__global__ void __launch_bounds__(kBlock)
k_bricks(const BrickEntry* __restrict__ list, const uint64_t* __restrict__ list_total, BrickSrc<kGather> src,
         BrickOut out)
{
    constexpr int kW = kBlock / kWave;
    static_assert(kGroupRecs <= kW * kWaveRecs, "the workgroup's brick fits the waves' buffers");
    __shared__ uint4 buf[kW * kWaveRecs];
    __shared__ uint32_t tab[kW][kTab];
    __shared__ uint32_t tot[kW];
    const uint32_t nl = (uint32_t)(*list_total >> 32);
    const uint32_t wv = uniform32(threadIdx.x / kWave);
    for (uint32_t l0 = blockIdx.x * kW; l0 < nl; l0 += gridDim.x * kW) {
        if (l0 + wv < nl) {
            const BrickEntry e = list[l0 + wv];
            if (e.z <= kWaveRecs)
                brick_in_lds<kWave, kWaveRecs / kWave, kGather>((uint32_t)__lane_id(), e, src, buf + wv * kWaveRecs,
                                                                tab[wv], nullptr, out);
        }
        for (uint32_t k = 0; k < kW && l0 + k < nl; ++k) {
            const BrickEntry e = list[l0 + k];
            if (e.z <= kWaveRecs || e.z > kGroupRecs) continue;   // workgroup-uniform
            __syncthreads();
            brick_in_lds<kBlock, kGroupRecs / kBlock, kGather>(threadIdx.x, e, src, buf, tab[0], tot, out);
        }
        __syncthreads();
    }
}

// One brick of any size by a workgroup, in memory: records grouped by key in
// the output range (w: pool index, or low key), each one's final place
// found from there and noted in the brick's source range, then the output
// written from the noted order.
template <int kT, bool kGather>
__device__ void brick_in_memory(const BrickEntry& e, const BrickSrc<kGather>& src, uint32_t* off, uint32_t* cur,
                                uint32_t* rank, uint64_t* tot, const BrickOut& out)
{
    const uint32_t t = threadIdx.x, n = e.z, base_rank = e.w;
    const uint64_t o = e.y;
    uint4* const buf = out.frag + o;
    for (uint32_t k = t; k < kTab; k += kT) off[k] = 0;
    __syncthreads();
    for (uint32_t i = t; i < n; i += kT) atomicAdd(off + (src.low(o + i) & (kBrickKeys - 1)), 1u);
    __syncthreads();
    static_assert(kT >= (int)kBrickKeys, "one key per thread");
    const uint32_t c = t < kBrickKeys ? off[t] : 0u;
    const uint64_t s = (uint64_t)c | ((uint64_t)(c != 0) << 32);
    const uint64_t p = group_incl_scan<kT>(s, tot) - s;
    __syncthreads();
    if (t < kBrickKeys) {
        off[t] = cur[t] = (uint32_t)p;
        rank[t] = (uint32_t)(p >> 32);
        if (c) out.row((uint64_t)base_rank + rank[t], e.x, t, (uint32_t)o + off[t], c);
        if (t + 1 == kBrickKeys) off[kBrickKeys] = n;
    }
    __syncthreads();
    for (uint32_t i = t; i < n; i += kT) {
        uint4 r;
        uint32_t low;
        if (kGather) {
            const uint2 ix = src.ent[o + i];
            r = src.pool[ix.x];
            r.w = ix.x;
            low = ix.y;
        } else {
            r = src.stage[o + i];
            low = r.w & (kBrickKeys - 1);
        }
        buf[atomicAdd(cur + low, 1u)] = r;
    }
    __threadfence();
    __syncthreads();
    for (uint32_t q = t; q < n; q += kT) {
        const uint4 x = buf[q];
        uint32_t leaf = 0;   // the last key whose run starts at or before q
#pragma unroll
        for (uint32_t d = kBrickKeys / 2; d >= 1; d >>= 1)
            if (off[leaf + d] <= q) leaf += d;
        const uint32_t lo = off[leaf], hi = off[leaf + 1];
        uint32_t before = 0;
        for (uint32_t d = lo; d < hi; ++d) before += rec_before(buf[d], d, x, q) ? 1u : 0u;
        if (kGather)
            src.ent[o + lo + before] = make_uint2(x.w, leaf);
        else
            src.stage[o + lo + before] = make_uint4(x.x, x.y, x.z, base_rank + rank[leaf]);
    }
    __threadfence();
    __syncthreads();
    for (uint32_t i = t; i < n; i += kT) {
        if (kGather) {
            const uint2 ix = src.ent[o + i];
            uint4 r = src.pool[ix.x];
            r.w = base_rank + rank[ix.y];
            buf[i] = r;
        } else {
            buf[i] = src.stage[o + i];
        }
    }
}

// Bricks above kGroupRecs records, found up to 64 list entries at a time: a
// workgroup takes one entry where the list is short (575 such bricks among
// 2,081 took 162 us in the 33 workgroups that 64 entries each make, 27 among
// 32 as long in one), and a part of 64 of a long list, most of whose bricks
// are small.
constexpr int kLargeBlock = 1024;

template <bool kGather>
__global__ void __launch_bounds__(kLargeBlock)
k_bricks_large(const BrickEntry* __restrict__ list, const uint64_t* __restrict__ list_total, BrickSrc<kGather> src,
               BrickOut out)
{
    __shared__ uint4 buf[kLdsRecs];
    __shared__ uint32_t off[kTab], cur[kTab], rank[kTab];
    __shared__ uint64_t tot[kLargeBlock / kWave];
    const uint32_t nl = (uint32_t)(*list_total >> 32);
    const uint32_t lane = (uint32_t)__lane_id();
    const uint32_t share = (nl + gridDim.x - 1) / gridDim.x, part = share < kWave ? share : kWave;
    for (uint32_t l0 = blockIdx.x * part; l0 < nl; l0 += gridDim.x * part) {
        uint64_t todo = __ballot(lane < part && l0 + lane < nl && list[l0 + lane].z > kGroupRecs);
        for (; todo; todo &= todo - 1) {   // the same in every wave
            const BrickEntry e = list[l0 + (uint32_t)__builtin_ctzll(todo)];
            if (e.z <= kLdsRecs)
                brick_in_lds<kLargeBlock, kLdsRecs / kLargeBlock, kGather>(threadIdx.x, e, src, buf, off,
                                                                           (uint32_t*)tot, out);
            else
                brick_in_memory<kLargeBlock, kGather>(e, src, off, cur, rank, tot, out);
            __syncthreads();
        }
    }
}

// Scan helpers. Bricks are scanned on (count | occupied << 32): the low
// half of the exclusive prefix is the brick's fragment offset, the high half
// its position in the list of occupied bricks.
struct LoadBrick {
    const uint32_t* cnt;
    __device__ uint64_t operator()(uint64_t i) const
    {
        const uint32_t c = cnt[i];
        return (uint64_t)c | ((uint64_t)(c != 0u) << 32);
    }
};

struct StoreBrick {
    uint32_t* off;
    BrickEntry* list;
    uint64_t n_list;   // entries it holds (fewer than bricks are occupied only where the arrays are too small)
    __device__ void operator()(uint64_t i, uint64_t v, uint64_t ex) const
    {
        off[i] = (uint32_t)ex;
        if ((uint32_t)v && (ex >> 32) < n_list) list[ex >> 32] = make_uint4((uint32_t)i, (uint32_t)ex, (uint32_t)v, 0u);
    }
};

// Distinct keys of the list's entries, replaced by their exclusive sums (the
// thread that stores an entry is the one that read it).
struct LoadOcc {
    const BrickEntry* list;
    const uint64_t* list_total;
    __device__ uint64_t operator()(uint64_t i) const { return i < (*list_total >> 32) ? list[i].w : 0u; }
};

struct StoreRank {
    BrickEntry* list;
    const uint64_t* list_total;
    __device__ void operator()(uint64_t i, uint64_t, uint64_t ex) const
    {
        if (i < (*list_total >> 32)) list[i].w = (uint32_t)ex;
    }
};

}  // namespace

struct CompactWs {
    uint32_t *brick_cnt, *brick_cur, *brick_off;
    BrickEntry* list;       // occupied bricks, ascending
    uint64_t* part;         // scan scratch
    uint64_t* list_total;   // (fragments | occupied bricks << 32)
    uint4* stage;           // two-pass capture and outputs over the pool: records
    uint2* ent;             // lists: (pool index, low key) by brick, and
    uint32_t* place;        //        each slot's place in its brick, in the same memory
};

static CompactWs carve_compact(void* ws, uint64_t n_head, uint64_t capacity, size_t* bytes)
{
    const uint64_t n_brick = (n_head + kBrickKeys - 1) / kBrickKeys;
    Carver c{(char*)ws, 0};
    CompactWs w;
    // adjacent, so that one fill clears both
    w.brick_cnt = c.take<uint32_t>(2 * n_brick);
    w.brick_cur = w.brick_cnt ? w.brick_cnt + n_brick : nullptr;
    w.brick_off = c.take<uint32_t>(n_brick);
    w.list = c.take<BrickEntry>(n_brick < capacity ? n_brick : capacity);
    w.part = c.take<uint64_t>(scan_scratch(n_brick));
    w.list_total = c.take<uint64_t>(1);
    w.stage = c.take<uint4>(capacity);
    w.ent = (uint2*)w.stage;
    w.place = w.ent ? (uint32_t*)(w.ent + capacity) : nullptr;
    if (bytes) *bytes = c.off + 256;
    return w;
}

size_t compact_ws_bytes(const fhv_capture_desc* d, uint64_t n_head, uint64_t capacity)
{
    (void)d;
    size_t b = 0;
    carve_compact(nullptr, n_head, capacity, &b);
    // callers size their buffers by 16 bytes per slot and a bit per key: the
    // query and the check both stay at that where less is used
    return std::max(b, (size_t)capacity * 16 + (size_t)(n_head / 8));
}

// Offsets of the bricks and the list of the occupied ones, from the counts.
static hipError_t brick_offsets(const CompactWs& w, uint64_t n_brick, uint64_t n_list, hipStream_t s)
{
    return scan<uint64_t>(LoadBrick{w.brick_cnt}, StoreBrick{w.brick_off, w.list, n_list}, n_brick, w.part, w.list_total, s);
}

// Ranks of the occupied bricks' first keys (and their number), after their
// fragments have been scattered or staged.
template <bool kGather>
static hipError_t brick_ranks(const Device& dev, const CompactWs& w, const BrickSrc<kGather>& src, uint64_t n_list,
                              uint64_t* n_occ, hipStream_t s)
{
    const uint64_t g = (n_list + kBlock / kWave - 1) / (kBlock / kWave), gmax = (uint64_t)dev.cus * 32;
    k_brick_occ<kGather><<<dim3((unsigned)(g < 1 ? 1 : g > gmax ? gmax : g)), dim3(kBlock), 0, s>>>(
        w.list, w.list_total, src);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return scan<uint64_t>(LoadOcc{w.list, w.list_total}, StoreRank{w.list, w.list_total}, n_list < 1 ? 1 : n_list,
                          w.part, n_occ, s);
}

// Per-brick sorts into the output arrays.
template <bool kGather>
static hipError_t brick_sorts(const Device& dev, const CompactWs& w, const BrickSrc<kGather>& src,
                              const fhv_pofa* out, uint64_t n_list, uint64_t capacity, const char* name,
                              hipStream_t s)
{
    ProfScope ps(dev, name, s);
    const BrickOut bo{(uint4*)out->frag, out->oct_key, out->oct_off, out->oct_cnt, out->cap_occ};
    const uint64_t g = (n_list + kBlock / kWave - 1) / (kBlock / kWave), gmax = (uint64_t)dev.cus * 32;
    k_bricks<kGather><<<dim3((unsigned)(g < 1 ? 1 : g > gmax ? gmax : g)), dim3(kBlock), 0, s>>>(w.list, w.list_total,
                                                                                              src, bo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || capacity <= kGroupRecs) return e;   // no brick can be larger
    k_bricks_large<kGather><<<dim3((unsigned)std::min<uint64_t>(n_list, (uint64_t)dev.cus)), dim3(kLargeBlock), 0, s>>>(
        w.list, w.list_total, src, bo);
    return hipGetLastError();
}

// Whether an output of the sorts shares memory with the pool they read.
static bool writes_pool(const fhv_lists* L, const fhv_pofa* out)
{
    const uintptr_t p0 = (uintptr_t)L->pool, p1 = p0 + 16 * L->capacity;
    const auto meets = [&](const void* q, uint64_t bytes) { return (uintptr_t)q < p1 && p0 < (uintptr_t)q + bytes; };
    const uint64_t rows = std::min(out->cap_occ, L->capacity);   // rows that can be written
    return meets(out->frag, 16 * L->capacity) || meets(out->oct_key, 8 * rows) || meets(out->oct_off, 4 * rows) ||
           meets(out->oct_cnt, 4 * rows);
}

hipError_t compact_launch(const Device& dev, const fhv_lists* L, const fhv_capture_desc* d,
                          const fhv_pofa* out, void* ws, hipStream_t s)
{
    (void)d;
    const uint64_t n_brick = (L->n_head + kBrickKeys - 1) / kBrickKeys;
    const uint64_t n_list = n_brick < L->capacity ? n_brick : L->capacity;   // occupied bricks at most
    CompactWs w = carve_compact(ws, L->n_head, L->capacity, nullptr);
    const bool wide = L->n_head > (1ull << 32);
    const bool in_place = writes_pool(L, out);
    hipError_t e;
    const uint64_t gmax = (uint64_t)dev.cus * 16;
    const auto grid = [&](uint64_t per) {
        const uint64_t g = (L->capacity + per - 1) / per;
        return dim3((unsigned)(g < 1 ? 1 : (g > gmax ? gmax : g)));
    };
    {
        ProfScope ps(dev, "compact.hist", s);
        e = fill_u32(w.brick_cnt, (in_place ? 2 : 1) * n_brick, 0u, s);
        if (e != hipSuccess) return e;
        if (wide)
            k_hist<uint64_t><<<grid((uint64_t)kBlock * kHistPer), dim3(kBlock), 0, s>>>(
                (const uint64_t*)L->keys, L->counter, L->capacity, w.brick_cnt, w.place, out->n_frag);
        else
            k_hist<uint32_t><<<grid((uint64_t)kBlock * kHistPer), dim3(kBlock), 0, s>>>(
                (const uint32_t*)L->keys, L->counter, L->capacity, w.brick_cnt, w.place, out->n_frag);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    {
        ProfScope ps(dev, "compact.scan", s);
        e = brick_offsets(w, n_brick, n_list, s);
    }
    if (e != hipSuccess) return e;
    if (in_place) {
        {
            ProfScope ps(dev, "compact.scatter", s);
            if (wide)
                k_stage<uint64_t><<<grid(kBlock), dim3(kBlock), 0, s>>>(
                    (const uint4*)L->pool, (const uint64_t*)L->keys, L->counter, L->capacity, w.brick_off, w.brick_cur,
                    w.stage);
            else
                k_stage<uint32_t><<<grid(kBlock), dim3(kBlock), 0, s>>>(
                    (const uint4*)L->pool, (const uint32_t*)L->keys, L->counter, L->capacity, w.brick_off, w.brick_cur,
                    w.stage);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
        const BrickSrc<false> src{nullptr, nullptr, w.stage};
        {
            ProfScope ps(dev, "compact.scan", s);
            e = brick_ranks(dev, w, src, n_list, out->n_occ, s);
        }
        if (e != hipSuccess) return e;
        return brick_sorts(dev, w, src, out, n_list, L->capacity, "compact.brick", s);
    }
    {
        ProfScope ps(dev, "compact.scatter", s);
        if (wide)
            k_scatter<uint64_t><<<grid(kBlock), dim3(kBlock), 0, s>>>(
                (const uint64_t*)L->keys, L->counter, L->capacity, w.brick_off, w.place, w.ent);
        else
            k_scatter<uint32_t><<<grid(kBlock), dim3(kBlock), 0, s>>>(
                (const uint32_t*)L->keys, L->counter, L->capacity, w.brick_off, w.place, w.ent);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    const BrickSrc<true> src{(const uint4*)L->pool, w.ent, nullptr};
    {
        ProfScope ps(dev, "compact.scan", s);
        e = brick_ranks(dev, w, src, n_list, out->n_occ, s);
    }
    if (e != hipSuccess) return e;
    return brick_sorts(dev, w, src, out, n_list, L->capacity, "compact.brick", s);
}

// Two-pass capture into arrays: after the count pass and the scans, the
// fragment total decides whether the arrays hold them; if not, only the
// counts are reported and the insert pass and the sorts do nothing. The
// bricks' 32-bit counts and their sum give the total modulo 2^32; `large`
// counts the passes that may have more, all others together have fewer than
// 2^32.
__global__ void k_arrays_check(uint64_t* __restrict__ list_total, const unsigned long long* __restrict__ large,
                               uint64_t capacity, uint64_t* __restrict__ n_frag, uint32_t* __restrict__ skip)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const uint64_t total = *large + (uint32_t)((uint32_t)*list_total - (uint32_t)*large);
    *n_frag = total;
    if (total > capacity) {
        *skip = 1u;
        *list_total = 0;   // no occupied bricks left to rank or sort
    } else {
        *skip = 0u;
    }
}

size_t capture_arrays_ws_bytes(const fhv_capture_desc* d, uint32_t n_tri, uint64_t capacity)
{
    const size_t cap_b = (capture_ws_bytes(d, n_tri) + 255) & ~(size_t)255;
    size_t b = 0;
    carve_compact(nullptr, 1ull << (3 * d->levels), capacity, &b);
    return cap_b + ((b + 255) & ~(size_t)255) + 256;
}

hipError_t capture_arrays_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d,
                                 const fhv_pofa* out, void* ws, hipStream_t s)
{
    const uint64_t n_head = 1ull << (3 * d->levels);
    const uint64_t n_brick = (n_head + kBrickKeys - 1) / kBrickKeys;
    const size_t cap_b = (capture_ws_bytes(d, m->n_tri) + 255) & ~(size_t)255;
    size_t cmp_b = 0;
    CompactWs w = carve_compact((char*)ws + cap_b, n_head, out->cap_frag, &cmp_b);
    uint32_t* skip = (uint32_t*)((char*)ws + cap_b + ((cmp_b + 255) & ~(size_t)255));
    unsigned long long* large = (unsigned long long*)(((uintptr_t)skip + 15) & ~(uintptr_t)7);
    const uint64_t n_list = n_brick < out->cap_frag ? n_brick : out->cap_frag;   // occupied bricks at most
    hipError_t e;
    {
        ProfScope ps(dev, "arrays.reset", s);
        e = fill_u32(w.brick_cnt, 2 * n_brick, 0u, s, (uint64_t*)large);
    }
    if (e != hipSuccess) return e;
    BrickSink bs{w.brick_cnt, w.brick_off, w.brick_cur, w.stage, skip, large};
    e = capture_bricks_launch(dev, m, d, ws, kActCount, bs, false, s);
    if (e != hipSuccess) return e;
    {
        ProfScope ps(dev, "arrays.scan", s);
        e = brick_offsets(w, n_brick, n_list, s);
        if (e == hipSuccess) {
            k_arrays_check<<<dim3(1), dim3(64), 0, s>>>(w.list_total, large, out->cap_frag, out->n_frag, skip);
            e = hipGetLastError();
        }
    }
    if (e != hipSuccess) return e;
    e = capture_bricks_launch(dev, m, d, ws, kActInsert, bs, true, s);
    if (e != hipSuccess) return e;
    const BrickSrc<false> src{nullptr, nullptr, w.stage};
    {
        ProfScope ps(dev, "arrays.scan", s);
        e = brick_ranks(dev, w, src, n_list, out->n_occ, s);
    }
    if (e != hipSuccess) return e;
    return brick_sorts(dev, w, src, out, n_list, out->cap_frag, "arrays.brick", s);
}

}  // namespace fhv
