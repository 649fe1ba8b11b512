// Embedding-layer simultaneous per-example gradient norms (Appendix B, embedding-layer algorithm) for gfx950:
//   w_b[v,d] = sum_{t: ids[b,t] = v} g[b,t,d]     (steps 1-2; the one-hot tensor and [B,V,D] are never formed)
//   s[b]     = sum_{v,d} w_b[v,d]^2               (step 3)
//   w'[v,d]  = sum_b w_b[v,d]                     (step 4)
// The positions p = b*T + t are sorted by id (stable, so positions ascend inside an id and the rows of one
// example are adjacent): a "segment" is all positions of one id, a "run" those of one id in one example, a
// "piece" at most kPiece consecutive sorted positions of one run (a run is cut wherever the sorted index is a
// multiple of kPiece).  Kernel A reads g, every row once, and fills the rows of w' that no id selects.  An id of at
// most kShort positions is finished there by one wave (each run's share of step 3, the row of w'), and so is an id of up
// to 64, by a wave that looks after nothing else but such ids.  A longer id is handed out piece by piece: a piece that is
// a whole run yields that run's share at once, the piece sums are parked in the workspace, and kernel B adds the
// parked sums in sorted order, an id of more than a thousand positions in parts shared out over workgroups.  However
// skewed the ids are, a wave of kernel A reads at most kChunk + kPiece rows, or those of the ids of 13 to 64 positions that
// begin in its 16; no floating-point number is added atomically: results are bitwise reproducible.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <type_traits>
#include <rocprim/device/device_radix_sort.hpp>

#include "../../include/lnpegn.h"
#include "lnpegn_device.h"

namespace lnpegn {
int g_emb_run_blocks = 4096;        // workgroups of kernel A per column group (each loops over its chunks)
namespace {

constexpr int kColBlock = 512;      // columns per wave: 8 per lane
constexpr int kChunk = 16;          // sorted positions whose piece heads one wave looks after
constexpr int kPiece = 32;          // longest piece; kChunk + kPiece + 1 lanes of one 64-lane window cover a wave's work
constexpr int kWavesPerBlock = 4;
constexpr int kNormBlocks = 2048;   // workgroups of the ||w'||^2 pass in accumulate mode
constexpr int kFillBlocks = 16384;  // most workgroups of the zero fill
constexpr int64_t kFillLeast = 8 << 10, kFillMost = 32 << 10;   // bytes that a wave of it takes at a time
constexpr int64_t kFillLateBytes = 40 << 20, kFillLateLarge = 128 << 20;   // most bytes of it that are left to kernel B

__global__ __launch_bounds__(256) void emb_prepare_kernel(const void *ids, int ids_i64, uint32_t *keys,
                                                          uint32_t *vals, int64_t n, int V)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        const int64_t id = ids_i64 ? static_cast<const int64_t *>(ids)[i] : (int64_t) static_cast<const int32_t *>(ids)[i];
        keys[i] = (id >= 0 && id < V) ? (uint32_t)id : (uint32_t)V;    // out of range: sorted behind, skipped
        vals[i] = (uint32_t)i;
    }
}

// ---------------------------------------------------------------------------------------
// Sort of the (id, position) pairs for batches of up to kSortTiles * kSortTile positions, in two launches.
// A pair travels as one word whose order is that of (id, position), so any correct sort of the words is the stable
// sort by id.  (1) Every workgroup sorts one tile of kSortTile words.  (2) The place of a word in the whole order is
// its index in its own tile plus the number of words below it in every other, found by binary search.
// Words are 32 bits (id, index within the tile) for vocabularies below 2^21 and 64 bits (id, position) beyond.
// ---------------------------------------------------------------------------------------
constexpr int kSortTile = 2048, kSortTileBits = 11;
constexpr int kSortTiles = 64;
constexpr int kSortEach = 4;                        // words per thread
constexpr int kSortThreads = kSortTile / kSortEach;
constexpr int kRankThreads = 256;

template <typename W>
struct SortWord;
template <>
struct SortWord<uint32_t> {
    static constexpr uint32_t kPad = ~0u;
    __device__ static uint32_t make(uint32_t key, uint32_t p) { return key << kSortTileBits | (p & (kSortTile - 1)); }
    __device__ static uint32_t key(uint32_t w) { return w >> kSortTileBits; }
    __device__ static uint32_t pos(uint32_t w, int tile) { return (uint32_t)tile * kSortTile + (w & (kSortTile - 1)); }
    // the least word of tile t that is not below w, a word of tile `mine`: positions of another tile are all below
    // or all above
    __device__ static uint32_t bound(uint32_t w, int t, int mine) { return (key(w) + (t < mine ? 1u : 0u)) << kSortTileBits; }
};
template <>
struct SortWord<uint64_t> {
    static constexpr uint64_t kPad = ~(uint64_t)0;
    __device__ static uint64_t make(uint32_t key, uint32_t p) { return (uint64_t)key << 32 | p; }
    __device__ static uint32_t key(uint64_t w) { return (uint32_t)(w >> 32); }
    __device__ static uint32_t pos(uint64_t w, int) { return (uint32_t)w; }
    __device__ static uint64_t bound(uint64_t w, int, int) { return w; }
};
__host__ __device__ inline bool sort_words_are_32(int V) { return V < (1 << (32 - kSortTileBits)) - 1; }

// the value of lane ^ kMask, without LDS memory
template <int kMask>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    const int i = (int)v;
    if constexpr (kMask == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xf, 0xf, true);       // quad_perm [1,0,3,2]
    else if constexpr (kMask == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
    else if constexpr (kMask == 4) {
        const int half = __builtin_amdgcn_update_dpp(0, i, 0x141, 0xf, 0xf, true);                            // row_half_mirror: ^ 7
        return (uint32_t)__builtin_amdgcn_update_dpp(0, half, 0x1B, 0xf, 0xf, true);                          // quad_perm [3,2,1,0]: ^ 3
    } else if constexpr (kMask == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0x128, 0xf, 0xf, true);   // row_ror:8
    else return (uint32_t)__shfl_xor(i, kMask, kWave);
}
template <int kMask>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v)
{
    return (uint64_t)lane_xor<kMask>((uint32_t)(v >> 32)) << 32 | lane_xor<kMask>((uint32_t)v);
}

// Zero fill beside the sort's second launch, a chain of a few workgroups' loads under which the memory idles: workgroup
// `block` clears kShadowBytes of w', whose first rows are cleared here whether their ids occur (kernel A writes those again)
// or not.  us a call, without / 32 MiB so / 48 MiB so / 12 beside the first launch and 32 beside the second: bf16 B=8 T=1024
// D=768 V=50257 47.3 / 46.0 / 46.6 / 45.7, B=16 T=2048 D=2048 124.6 / 118.5 / 118.0 / 118.1, B=16 T=512 D=1024 V=60000
// 63.0 / 58.2 / 58.1 / 57.6, B=16 T=1024 D=512 V=32000 49.0 / 49.6 / 49.3 / 49.1.
struct ShadowFill {
    float *begin;        // 16-byte aligned
    int64_t len;         // floats
    int blocks;          // workgroups
};
constexpr int kShadowBytes = 32 << 10;               // of a workgroup
constexpr int64_t kShadowMost = 32 << 20;            // in all
__device__ __forceinline__ void shadow_fill(const ShadowFill &f, int block)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    constexpr int kFloats = kShadowBytes / 4;
    const int64_t at = (int64_t)block * kFloats;
    const int len = (int)min((int64_t)kFloats, f.len - at), quads = len / 4;
    float *p = f.begin + at;
#pragma unroll 8
    for (int i = threadIdx.x; i < quads; i += kRankThreads) __builtin_nontemporal_store(f32x4{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<f32x4 *>(p) + i);
    if ((int)threadIdx.x < len - quads * 4) p[quads * 4 + threadIdx.x] = 0.f;
}

// Bitonic network over a tile, four consecutive words per thread: strides below 4 stay in a thread's registers, below
// 256 in the wave (DPP and lane permutes), and only the six stages of 256 and more go through LDS with a barrier.
// Bound by the chain of 66 stages: with every stage through LDS, one compare-exchange per thread, 16.4 us against
// 5.9 for 4 tiles.
template <typename W>
__global__ __launch_bounds__(kSortThreads) void emb_tile_sort_kernel(const void *ids, int ids_i64, int64_t n, int V, W *tiles)
{
    __shared__ __align__(16) W mem[kSortTile];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kSortTile + tid * kSortEach;
    W a[kSortEach];
#pragma unroll
    for (int e = 0; e < kSortEach; ++e) {
        const int64_t p = base + e;
        a[e] = SortWord<W>::kPad;
        if (p < n) {
            const int64_t id = ids_i64 ? static_cast<const int64_t *>(ids)[p] : (int64_t) static_cast<const int32_t *>(ids)[p];
            const uint32_t key = (id >= 0 && id < V) ? (uint32_t)id : (uint32_t)V;   // out of range: sorted behind, skipped
            a[e] = SortWord<W>::make(key, (uint32_t)p);
        }
    }
    auto in_order = [](W &x, W &y, bool ascending) {
        const W lo = x < y ? x : y, hi = x < y ? y : x;
        x = ascending ? lo : hi;
        y = ascending ? hi : lo;
    };
    auto keep = [](W mine, W other, bool low) { return low ? (mine < other ? mine : other) : (mine < other ? other : mine); };
    auto across = [&](auto mask, int k) {              // stride 4 * mask: lanes of one wave
        constexpr int kMask = decltype(mask)::value;
        const bool low = ((tid & kMask) == 0) == ((tid * kSortEach & k) == 0);
#pragma unroll
        for (int e = 0; e < kSortEach; ++e) a[e] = keep(a[e], lane_xor<kMask>(a[e]), low);
    };
    auto within = [&](int k) {                         // strides 2 and 1
        const bool up = (tid * kSortEach & k) == 0;
        in_order(a[0], a[2], up);
        in_order(a[1], a[3], up);
        in_order(a[0], a[1], up);
        in_order(a[2], a[3], up);
    };
    in_order(a[0], a[1], true);                        // k = 2
    in_order(a[2], a[3], false);
    within(4);
#pragma unroll
    for (int k = 8; k <= kSortTile; k <<= 1) {
        for (int j = k >> 1; j >= 256; j >>= 1) {      // strides beyond a wave
            __syncthreads();
#pragma unroll
            for (int e = 0; e < kSortEach; ++e) mem[tid * kSortEach + e] = a[e];
            __syncthreads();
            const bool low = ((tid * kSortEach & j) == 0) == ((tid * kSortEach & k) == 0);
#pragma unroll
            for (int e = 0; e < kSortEach; ++e) a[e] = keep(a[e], mem[(tid * kSortEach ^ j) + e], low);
        }
        if (k >= 256) across(std::integral_constant<int, 32>{}, k);
        if (k >= 128) across(std::integral_constant<int, 16>{}, k);
        if (k >= 64) across(std::integral_constant<int, 8>{}, k);
        if (k >= 32) across(std::integral_constant<int, 4>{}, k);
        if (k >= 16) across(std::integral_constant<int, 2>{}, k);
        across(std::integral_constant<int, 1>{}, k);
        within(k);
    }
#pragma unroll
    for (int e = 0; e < kSortEach; ++e) tiles[base + e] = a[e];
}

// Each thread places one word.  Every 32nd word of every tile is copied to LDS; sixteen binary searches (one per
// other tile) advance together, first over those samples, then inside the 32 words (one cache line of 32-bit words)
// that they leave.  Latency bound: with all eleven steps in memory 10.8 us for 16 tiles and 9.0 for 4, against 7.6
// and 6.9 (with whole tiles in LDS, which leaves one workgroup a CU, 14.0 and 6.9).
constexpr int kSampleEvery = 32, kSamples = kSortTile / kSampleEvery;
template <typename W>
__global__ __launch_bounds__(kRankThreads) void emb_rank_kernel(const W *tiles, int ntiles, int64_t n, uint32_t *sorted_ids,
                                                                uint32_t *sorted_pos, ShadowFill fill)
{
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int kPerTile = kSortTile / kRankThreads;
    if ((int)blockIdx.x >= ntiles * kPerTile) {
        shadow_fill(fill, (int)blockIdx.x - ntiles * kPerTile);
        return;
    }
    W *samples = reinterpret_cast<W *>(lds);                     // [ntiles][kSamples]: the last word of each block
    const int64_t i = (int64_t)blockIdx.x * kRankThreads + threadIdx.x;     // index into the tiles array
    const W word = tiles[i];                                     // (the grid covers the tiles exactly)
#pragma unroll 4
    for (int v = threadIdx.x; v < ntiles * kSamples; v += kRankThreads)
        samples[v] = tiles[(int64_t)v * kSampleEvery + kSampleEvery - 1];
    __syncthreads();
    if (word == SortWord<W>::kPad) return;
    const int mine = (int)(i / kSortTile);
    int64_t rank = i - (int64_t)mine * kSortTile;
    constexpr int kGroup = 16;
    for (int t0 = 0; t0 < ntiles; t0 += kGroup) {
        W bound[kGroup];
        int tile[kGroup], pos[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            tile[u] = min(t0 + u, ntiles - 1);                   // a tile that does not exist: searched, not counted
            bound[u] = SortWord<W>::bound(word, tile[u], mine);
            pos[u] = 0;
        }
        // blocks whose last word is below `bound`: branch-free lower bound over the 64 samples
#pragma unroll
        for (int step = kSamples / 2; step > 0; step >>= 1)
#pragma unroll
            for (int u = 0; u < kGroup; ++u)
                pos[u] += samples[tile[u] * kSamples + pos[u] + step - 1] < bound[u] ? step : 0;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            pos[u] += samples[tile[u] * kSamples + pos[u]] < bound[u] ? 1 : 0;
            pos[u] *= kSampleEvery;
        }
        // the words below it inside the next block (whose last word is not); none if there is no next block
#pragma unroll
        for (int step = kSampleEvery / 2; step > 0; step >>= 1)
#pragma unroll
            for (int u = 0; u < kGroup; ++u)
                pos[u] += tiles[tile[u] * kSortTile + min(pos[u] + step, kSortTile) - 1] < bound[u] && pos[u] < kSortTile ? step : 0;
#pragma unroll
        for (int u = 0; u < kGroup; ++u)
            if (t0 + u < ntiles && t0 + u != mine) rank += pos[u];
    }
    sorted_ids[rank] = SortWord<W>::key(word);
    sorted_pos[rank] = SortWord<W>::pos(word, mine);
}

// eight columns of one row, added into sub: 16-byte loads when the row allows, element loads otherwise
__device__ __forceinline__ void add_row(const bf16_t *g, int64_t p, int D, int c0, bool vec, float (&sub)[8])
{
    const bf16_t *row = g + p * D + c0;
    if (vec) {
        const uint4 r = *reinterpret_cast<const uint4 *>(row);
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sub[2 * i] += __builtin_bit_cast(float, w[i] << 16);
            sub[2 * i + 1] += __builtin_bit_cast(float, w[i] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (c0 + i < D) sub[i] += load_elem<bf16_t>(row, i);
    }
}

// the same eight columns as raw 16-byte loads, for callers that want several rows in flight
template <typename T>
struct Row8;
template <>
struct Row8<bf16_t> {
    uint4 a;
};
template <>
struct Row8<float> {
    float4 a, b;
};
__device__ __forceinline__ Row8<bf16_t> load_row8(const bf16_t *g, int64_t p, int D, int c0)
{
    return Row8<bf16_t>{*reinterpret_cast<const uint4 *>(g + p * D + c0)};
}
__device__ __forceinline__ Row8<float> load_row8(const float *g, int64_t p, int D, int c0)
{
    const float *row = g + p * D + c0;
    return Row8<float>{*reinterpret_cast<const float4 *>(row), *reinterpret_cast<const float4 *>(row + 4)};
}
__device__ __forceinline__ void unpack_row8(const Row8<bf16_t> &r, float (&f)[8])
{
    const uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __builtin_bit_cast(float, w[i] << 16);
        f[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void unpack_row8(const Row8<float> &r, float (&f)[8])
{
    f[0] = r.a.x; f[1] = r.a.y; f[2] = r.a.z; f[3] = r.a.w;
    f[4] = r.b.x; f[5] = r.b.y; f[6] = r.b.z; f[7] = r.b.w;
}

__device__ __forceinline__ void add_row(const float *g, int64_t p, int D, int c0, bool vec, float (&sub)[8])
{
    const float *row = g + p * D + c0;
    if (vec) {
        const float4 lo = *reinterpret_cast<const float4 *>(row), hi = *reinterpret_cast<const float4 *>(row + 4);
        sub[0] += lo.x; sub[1] += lo.y; sub[2] += lo.z; sub[3] += lo.w;
        sub[4] += hi.x; sub[5] += hi.y; sub[6] += hi.z; sub[7] += hi.w;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (c0 + i < D) sub[i] += row[i];
    }
}

// eight fp32 columns of a row: out[k] = (add ? row[k] : 0) + in[k], stored; returns the sum of squares
// stream: the row will not be read again soon (a row of w'): streaming stores, kept out of the caches
__device__ __forceinline__ float put_row(float *row, const float (&in)[8], int c0, int D, bool add, bool stream = false)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    float sq = 0.f;
    if (c0 + 8 <= D && (reinterpret_cast<uintptr_t>(row) & 15u) == 0) {
        float4 lo = make_float4(in[0], in[1], in[2], in[3]), hi = make_float4(in[4], in[5], in[6], in[7]);
        if (add) {
            const float4 a = *reinterpret_cast<const float4 *>(row), b = *reinterpret_cast<const float4 *>(row + 4);
            lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
            hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
        }
        if (stream) {
            __builtin_nontemporal_store(f32x4{lo.x, lo.y, lo.z, lo.w}, reinterpret_cast<f32x4 *>(row));
            __builtin_nontemporal_store(f32x4{hi.x, hi.y, hi.z, hi.w}, reinterpret_cast<f32x4 *>(row + 4));
        } else {
            *reinterpret_cast<float4 *>(row) = lo;
            *reinterpret_cast<float4 *>(row + 4) = hi;
        }
        sq = lo.x * lo.x + lo.y * lo.y + lo.z * lo.z + lo.w * lo.w + hi.x * hi.x + hi.y * hi.y + hi.z * hi.z + hi.w * hi.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (c0 + k < D) {
                const float v = add ? row[k] + in[k] : in[k];
                row[k] = v;
                sq = fmaf(v, v, sq);
            }
    }
    return sq;
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane)      // lane is wave-uniform
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// First index in [lo, lo + len] from which on the ascending values of `a` are not below target; every lane searches for
// its own target.  Seven probes a round: a third of the dependent loads.
__device__ __forceinline__ int64_t lower_bound_value(const uint32_t *a, int64_t lo, int64_t len, uint32_t target)
{
    while (__any(len > 0)) {
        const int64_t step = len / 8 + 1;              // probes at lo + step - 1, lo + 2 step - 1, ...
        uint32_t p[7];
#pragma unroll
        for (int u = 0; u < 7; ++u) p[u] = step * (u + 1) <= len ? a[lo + step * (u + 1) - 1] : 0xffffffffu;
        int below = 0;
#pragma unroll
        for (int u = 0; u < 7; ++u) below += (step * (u + 1) <= len && p[u] < target) ? 1 : 0;
        lo += step * below;
        len = len - step * below < step - 1 ? len - step * below : step - 1;
    }
    return lo;
}

// For each half of the wave, the first of its lo .. lo+len for which below(index) is false, where it is true up to there:
// 32 probes a round, the two halves side by side.
template <typename F>
__device__ __forceinline__ uint32_t half_wave_first_not(uint32_t lo, uint32_t len, int lane, F below)
{
    while (__any(len > 0)) {
        const uint32_t step = len / 33 + 1, at = step * ((lane & 31) + 1);      // probes at lo + step - 1, lo + 2 step - 1, ...
        const uint64_t yes = __ballot(at <= len && below(lo + min(at, len) - 1));
        const uint32_t c = __builtin_popcount((uint32_t)(lane < 32 ? yes : yes >> 32));
        lo += step * c;
        len = min(len - step * c, step - 1);
    }
    return lo;
}

// Zero fill of the rows of w' that no id selects (rows begin to end - 1), a part of kernel A's grid and of kernel B's:
// the rows of ids that occur are written, whole, by the other workgroups, so everything touches different rows and
// runs side by side.  Kernel A waits for its chains of loads more than for bandwidth and kernel B does little else, so
// the fill is shared out between the two: half of it, at most 40 MiB, or of a large w' 128 MiB, beside kernel B
// (run_embedding).  A wave takes `rows` neighbouring
// rows (at most 64) and finds their ids in the sorted list, so that no map of the ids is needed before the launch;
// waves beside each other take rows beside each other, so that together they sweep one moving window of w'.  Absent rows
// in a row are one stretch of memory: whole lines but at its ends, whatever the width.  (A row at a time, a lane's
// search each, sixteen rows of which lay far apart / this, us a presorted call: B=8 T=1024 D=8 V=1000000 fp32 140 / 25,
// B=512 T=512 D=64 V=1000000 360 / 145, D=2344 V=240547 511 / 443, B=8 T=1024 D=768 V=50257 46 / 37.5.  By a map of the ids
// and a kernel of its own on a second stream: 54, 207, 408, 60.)
// Streaming stores: the zeros are not wanted in any cache (the rows read next are g's), and lines left dirty
// in the memory-side cache would be written back one by one under the reads that follow.
__device__ __forceinline__ void fill_absent_rows(const uint32_t *keys, uint32_t n, float *w, int begin, int end, int D, int rows,
                                                 int wave, int nwaves, int lane)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    for (int64_t r0 = begin + (int64_t)wave * rows; r0 < end; r0 += (int64_t)nwaves * rows) {
        const uint32_t first = (uint32_t)r0, behind = (uint32_t)(r0 + rows < end ? r0 + rows : end), target = lane < 32 ? first : behind;
        const uint32_t found = half_wave_first_not(0, n, lane, [&](uint32_t k) { return keys[k] < target; });
        const uint32_t q_begin = lane_value(found, 0), q_end = lane_value(found, 32);
        uint64_t absent = ~(uint64_t)0 >> (64 - (behind - first));
        if (q_end - q_begin <= 512) {                  // the ids that occur, one after the other
            for (uint32_t q = q_begin; q < q_end; q += 64) {
                const uint32_t key = q + lane < q_end ? keys[q + lane] : 0xffffffffu;
                const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, 0x138, 0xf, 0xf, false);   // wave_shr:1
                for (uint64_t ids = __ballot(key != before && key < behind); ids; ids &= ids - 1)
                    absent &= ~((uint64_t)1 << (lane_value(key, __builtin_ctzll(ids)) - first));
            }
        } else {                                       // ... or a search for each
            const uint32_t row = first + lane;
            const int64_t at = lower_bound_value(keys, q_begin, q_end - q_begin, row);
            absent &= ~__ballot(row < behind && at < q_end && keys[at] == row);
        }
        while (absent) {
            const int r = __builtin_ctzll(absent);
            const uint64_t others = ~(absent >> r);
            const int count = others ? __builtin_ctzll(others) : 64;
            absent &= count + r < 64 ? ~(uint64_t)0 << (count + r) : 0;
            float *p = w + (r0 + r) * D;
            const int64_t len = (int64_t)count * D;
            const int head = (int)(min((int64_t)((16 - (reinterpret_cast<uintptr_t>(p) & 15u)) & 15u) / 4, len));
            const int64_t quads = (len - head) / 4;
            if (lane < head) p[lane] = 0.f;
            for (int64_t i = lane; i < quads; i += 64)
                __builtin_nontemporal_store(f32x4{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<f32x4 *>(p + head) + i);
            if (lane < len - head - quads * 4) p[head + quads * 4 + lane] = 0.f;
        }
    }
}

// Kernel A.  keys/vals: positions sorted by id.  A segment is short (at most kShort positions), medium (at most 64)
// or long.  The waves of the runs look after kChunk sorted positions each: a short segment belongs whole to the wave
// whose positions hold its first one, and that wave finishes the id (every run's share of s[b], the row of w').
// A long segment is handed out piece by piece to the waves whose positions hold the pieces' first rows; a piece that is
// a whole run yields that run's share of s[b], and every sum is parked.  Medium segments are finished the same way
// as short ones, by waves of their own that see 64 positions from the segment's first (cut into pieces and parked
// too, they added a fifth to the traffic of B=16 T=2048 D=2048; with kernel B left to the long ones 129 -> 127 us, and
// B=64 T=512 D=1024 fp32 106 -> 91).
// A wave of the runs sees kShort positions back (to tell whether a piece in its chunk belongs to a short segment that
// an earlier wave owns) and far enough ahead for anything that starts in its chunk; rows are streamed sixteen
// (fp32: eight) at a time.  contrib [ncb][n]: a run's share of s[b], at the run's first position (from
// kernel B: at another of the run's), zero elsewhere;
// bigpart [ncb][n]: squared norm of a finished row of w', at the segment's first position (not when accumulating),
// zero elsewhere.  The zeros are written by the waves of the runs, so neither array is cleared before; also where kernel B
// puts a norm afterwards.  arrived [n / part + 1][ncb] (part = 1 << part_bits): kernel B's counters, cleared here.
// runsum [n][D]: parked sums, at the piece's first position.
constexpr int kShort = 12;
static_assert(kShort + kChunk + kPiece < 63 && kShort + kChunk + kShort < 63, "one 64-lane window must cover a wave's work");

// Sums over the wave of eight values per lane at once: lane j's result is the sum of a[j & 7].  Three steps halve
// the values and the lanes they are spread over together, so eight sums cost little more than two.
__device__ __forceinline__ float wave_sums8(const float (&a)[8], int lane)
{
    float b[4], c[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float keep = lane & 1 ? a[2 * i + 1] : a[2 * i], send = lane & 1 ? a[2 * i] : a[2 * i + 1];
        b[i] = keep + __builtin_bit_cast(float, lane_xor<1>(__builtin_bit_cast(uint32_t, send)));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = lane & 2 ? b[2 * i + 1] : b[2 * i], send = lane & 2 ? b[2 * i] : b[2 * i + 1];
        c[i] = keep + __builtin_bit_cast(float, lane_xor<2>(__builtin_bit_cast(uint32_t, send)));
    }
    const float keep = lane & 4 ? c[1] : c[0], send = lane & 4 ? c[0] : c[1];
    float d = keep + __builtin_bit_cast(float, lane_xor<4>(__builtin_bit_cast(uint32_t, send)));
    d += __builtin_bit_cast(float, lane_xor<8>(__builtin_bit_cast(uint32_t, d)));
    d += __builtin_bit_cast(float, lane_xor<16>(__builtin_bit_cast(uint32_t, d)));
    d += __builtin_bit_cast(float, lane_xor<32>(__builtin_bit_cast(uint32_t, d)));
    return d;
}

// What becomes of the rows of a window (one sorted position per lane), as masks over the lanes.
struct RowEnds {
    uint64_t close;      // last row of a run or piece: its sum is complete
    uint64_t id;         // ... and the last row of its id: the row of w' is
    uint64_t park;       // ... of a piece: its sum is parked
    uint64_t whole;      // ... of a whole run: its squared norm is its share of s[b]
    uint32_t head_pos;   // per lane: position of the first row of this row's run or piece
    uint32_t id_pos;     // per lane: position of the first row of this row's id
};

// Adds up rows l .. e-1 of the window (l starts a run or piece, e-1 ends one), for one column block.  Bound by its
// instructions: about 200 a row when the rows were taken one at a time out of a register array, with a reduction
// over the wave at every end; unrolled, with the ends of eight rows reduced together, kernel A
// alone takes 14.8 us instead of 18.7 at B=8 T=1024 D=768 and 59 instead of 68 at B=16 T=2048 D=2048.
template <typename T, bool kVec>
__device__ __forceinline__ void stream_rows(const T *g, float *w, float *runsum, float *contrib, float *bigpart, int64_t n, int D,
                                            int accumulate, int cb, int lane, uint32_t key, uint32_t val, int l, int e,
                                            const RowEnds &ends)
{
    constexpr int kRows = kVec && sizeof(T) == 2 ? 16 : 8;       // rows in flight
    const int c0 = cb * kColBlock + lane * 8;
    const bool has_cols = c0 < D;
    const int c_load = has_cols ? c0 : 0;                        // lanes without columns fetch what lane 0 does
    float sub[8], tot[8];                // the open run or piece; the id's runs so far
#pragma unroll
    for (int k = 0; k < 8; ++k) sub[k] = tot[k] = 0.f;
    for (int r = l; r < e; r += kRows) {
        // the loads carry no condition (a row past the end repeats the last one and is dropped afterwards), so that
        // all are issued before the first is waited for
        Row8<T> raw[kVec ? kRows : 1];
        float part[kVec ? 1 : kRows][8];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            if constexpr (kVec) {
                raw[u] = load_row8(g, (int64_t)lane_value(val, min(r + u, e - 1)), D, c_load);
            } else {                                             // ragged or unaligned columns: element loads
#pragma unroll
                for (int k = 0; k < 8; ++k) part[u][k] = 0.f;
                if (has_cols && r + u < e) add_row(g, (int64_t)lane_value(val, r + u), D, c0, false, part[u]);
            }
        }
#pragma unroll
        for (int h = 0; h < kRows; h += 8) {
            float sq[8], wsq[8];                                 // squared norms that rows r+h .. r+h+7 complete
#pragma unroll
            for (int u = 0; u < 8; ++u) sq[u] = wsq[u] = 0.f;
            auto row = [&](int u, float (&f)[8]) {
                if constexpr (kVec) {
                    unpack_row8(raw[h + u], f);
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k) f[k] = part[h + u][k];
                }
            };
            auto add = [&](int u, const float (&f)[8]) {
                const int t = r + h + u;
#pragma unroll
                for (int k = 0; k < 8; ++k) sub[k] += f[k];
                if ((ends.close >> t) & 1) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) sq[u] = fmaf(sub[k], sub[k], sq[u]);
                    if (!has_cols) sq[u] = 0.f;                  // such lanes hold a copy of lane 0's columns
                    if ((ends.park >> t) & 1) {
                        if (has_cols) put_row(runsum + (int64_t)lane_value(ends.head_pos, t) * D + c0, sub, c0, D, false);
                    } else {
#pragma unroll
                        for (int k = 0; k < 8; ++k) tot[k] += sub[k];
                        if ((ends.id >> t) & 1) {
                            if (has_cols)
                                wsq[u] = put_row(w + (int64_t)lane_value(key, t) * D + c0, tot, c0, D, accumulate != 0, true);
#pragma unroll
                            for (int k = 0; k < 8; ++k) tot[k] = 0.f;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) sub[k] = 0.f;
                }
            };
            // Eight rows of one run or piece are added as a tree, which rounds less than one after the other (the parked
            // sums of a long id cancel) and checks nothing in between.
            float all[8];
            int from = 0;
            if (r + h + 7 < e && !(ends.close >> (r + h) & 0x7f)) {
                float f2[8], f3[8];
                auto pair = [&](int u, float (&to)[8]) {
                    float next[8];
                    row(u, to);
                    row(u + 1, next);
#pragma unroll
                    for (int k = 0; k < 8; ++k) to[k] += next[k];
                };
                pair(0, all);
                pair(2, f2);
#pragma unroll
                for (int k = 0; k < 8; ++k) all[k] += f2[k];
                pair(4, f2);
                pair(6, f3);
#pragma unroll
                for (int k = 0; k < 8; ++k) all[k] += f2[k] + f3[k];
                from = 7;
            } else {
                row(7, all);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (r + h + u < e && u >= from) {
                    float f[8];
                    if (u < 7) row(u, f);
                    if (u < 7) add(u, f);
                    else add(u, all);
                }
            }
            const int t = r + h + (lane & 7);                    // lane j < 8 stores what row r+h+j completed
            if (r + h < e && (ends.close >> (r + h) & 0xff)) {
                const float total = wave_sums8(sq, lane);
                const uint32_t at = (uint32_t)__shfl((int)ends.head_pos, t & 63);
                if (lane < 8 && t < e && ((ends.whole >> t) & 1)) contrib[(int64_t)cb * n + at] = total;
                if (!accumulate && (ends.id >> (r + h) & 0xff)) {
                    const float wtotal = wave_sums8(wsq, lane);
                    const uint32_t wat = (uint32_t)__shfl((int)ends.id_pos, t & 63);
                    if (lane < 8 && t < e && ((ends.id >> t) & 1)) bigpart[(int64_t)cb * n + wat] = wtotal;
                }
            }
        }
    }
}

// The medium segments whose first sorted position is among the kChunk from q0, for one column block.
template <typename T, bool kVec>
__device__ __forceinline__ void finish_medium_ids(const T *g, const uint32_t *keys, const uint32_t *vals, float *w, float *contrib,
                                                  float *bigpart, int64_t n, int Tn, int D, int V, int accumulate, int64_t q0, int cb,
                                                  int lane)
{
    const int64_t q = q0 + lane;
    const uint32_t key = q < n ? keys[q] : 0xffffffffu, before = q > 0 && q < n ? keys[q - 1] : 0xffffffffu;
    const uint32_t ahead = q + kShort < n ? keys[q + kShort] : 0xffffffffu, beyond = q + 64 < n ? keys[q + 64] : 0xffffffffu;
    for (uint64_t ids = __ballot(lane < kChunk && key < (uint32_t)V && key != before && ahead == key && beyond != key); ids; ids &= ids - 1) {
        const int64_t at = q0 + __builtin_ctzll(ids) + lane;
        const uint32_t k = at < n ? keys[at] : 0xffffffffu, p = at < n ? vals[at] : 0u, v = lane_value(k, 0);
        const uint32_t ex = p / (uint32_t)Tn, prev_ex = (uint32_t)__shfl_up((int)ex, 1);
        const uint64_t m_heads = __ballot(k == v && (lane == 0 || ex != prev_ex));
        const int len = __builtin_popcountll(__ballot(k == v));  // the low lanes
        RowEnds ends;
        ends.id = (uint64_t)1 << (len - 1);
        ends.close = ends.whole = m_heads >> 1 | ends.id;
        ends.park = 0;
        ends.head_pos = (uint32_t)__shfl((int)p, 63 - __builtin_clzll((m_heads & (((uint64_t)2 << lane) - 1)) | 1u));
        ends.id_pos = lane_value(p, 0);
        stream_rows<T, kVec>(g, w, nullptr, contrib, bigpart, n, D, accumulate, cb, lane, k, p, 0, len, ends);
    }
}

// kVec: every lane that has columns has eight whole ones behind an aligned 16-byte boundary (D % 8 == 0 and
// aligned rows); rows are then fetched as vectors, sixteen bf16 rows or eight fp32 rows in flight.
// Grid: medium_blocks workgroups for the medium segments (the longest chains, so first), then fill_blocks workgroups
// of the fill among runs_x times the groups of kWavesPerBlock column blocks.
template <typename T, bool kVec>
__global__ __launch_bounds__(64 * kWavesPerBlock, kVec && sizeof(T) == 2 ? 3 : 4) void emb_runs_kernel(
    const T *g, const uint32_t *keys, const uint32_t *vals, float *w, float *runsum, float *contrib, float *bigpart,
    uint32_t *arrived, int64_t n, int part_bits, int Tn, int D, int V, int accumulate, int medium_blocks, int fill_begin,
    int fill_end, int fill_each, int fill_blocks, int runs_x)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x < medium_blocks) {
        // the waves of a workgroup take the same positions and neighbouring column blocks
        const int column_groups = (D + kColBlock * kWavesPerBlock - 1) / (kColBlock * kWavesPerBlock);
        const int span = (int)blockIdx.x / column_groups, cb = ((int)blockIdx.x - span * column_groups) * kWavesPerBlock + wave;
        if (cb * kColBlock < D)
            finish_medium_ids<T, kVec>(g, keys, vals, w, contrib, bigpart, n, Tn, D, V, accumulate, (int64_t)span * kChunk, cb, lane);
        return;
    }
    // One workgroup of the fill after every two of the runs, then what is left of either: the runs, each a chain of
    // loads, must all be under way early, and the fill's stores go out beside them.
    const int run_blocks = (int)gridDim.x - medium_blocks - fill_blocks, groups = min(run_blocks / 2, fill_blocks);
    const int j = (int)blockIdx.x - medium_blocks, behind = j - 3 * groups;
    const int block = behind < 0 ? 2 * (j / 3) + j % 3 : 2 * groups + behind;
    int fill = behind < 0 && j % 3 == 2 ? j / 3 : -1;
    if (behind >= 0 && block >= run_blocks) fill = groups + block - run_blocks;
    if (fill >= 0) {
        fill_absent_rows(keys, (uint32_t)n, w, fill_begin, fill_end, D, fill_each, fill * kWavesPerBlock + wave, fill_blocks * kWavesPerBlock, lane);
        return;
    }
    const int block_y = block / runs_x, block_x = block - block_y * runs_x;
    // the waves of a workgroup take the same positions and neighbouring column blocks: a row of g is then
    // read whole by one workgroup at one time
    const int cb = block_y * kWavesPerBlock + wave;
    if (cb * kColBlock >= D) return;
    // A workgroup takes chunks block_x, block_x + runs_x, ...; the next chunk's part of the sorted list
    // is fetched while this chunk's rows are on their way.
    // Lane l looks at sorted position i0 - kShort - 1 + l: lane 0 only serves as "the position before",
    // lanes kShort+1 .. kShort+kChunk are the chunk.
    const int64_t nchunks = (n + kChunk - 1) / kChunk;
    // far, near: the keys 64 positions ahead and back, which tell medium segments from long ones.
    auto look = [&](int64_t chunk, uint32_t &k, uint32_t &p, uint32_t &far, uint32_t &near) {
        const int64_t q = chunk * kChunk - kShort - 1 + lane;
        const bool in = chunk < nchunks && q >= 0 && q < n;
        k = in ? keys[q] : 0xffffffffu;
        p = in ? vals[q] : 0u;
        far = in && q + 64 < n ? keys[q + 64] : 0xffffffffu;
        near = chunk < nchunks && q >= 64 ? keys[q - 64 < n ? q - 64 : 0] : 0xffffffffu;
    };
    uint32_t key_next, val_next, far_next, near_next;
    look(block_x, key_next, val_next, far_next, near_next);
    for (int64_t chunk = block_x; chunk < nchunks; chunk += runs_x) {
    const int64_t i0 = chunk * kChunk;
    const int64_t q = i0 - kShort - 1 + lane;
    const uint32_t key = key_next, val = val_next, far = far_next, near = near_next;
    look(chunk + runs_x, key_next, val_next, far_next, near_next);
    const uint32_t ex = val / (uint32_t)Tn;
    const uint32_t pkey = (uint32_t)__shfl_up((int)key, 1), pex = (uint32_t)__shfl_up((int)ex, 1);
    const bool valid = key < (uint32_t)V;
    const uint64_t m_valid = __ballot(valid);
    const uint64_t m_head = __ballot(valid && lane >= 1 && (key != pkey || ex != pex));     // starts a run
    const uint64_t m_seg = __ballot(valid && lane >= 1 && key != pkey);                     // starts a segment
    const uint64_t m_piece = m_head | __ballot(valid && lane >= 1 && q % kPiece == 0);      // starts a piece
    // is this lane's segment more than short?  Its first position is the nearest segment head at or below the lane
    // (not in the window: it lies more than kShort back), its end the next segment head or invalid key
    // (not in the window: more than kShort ahead of anything this wave may own).
    const uint64_t upto = ((uint64_t)2 << lane) - 1, m_ends = m_seg | ~m_valid;
    const uint64_t heads_below = m_seg & upto, ends_above = m_ends & ~upto;
    const int seg_first = heads_below ? 63 - __builtin_clzll(heads_below) : -1;
    const int seg_end = ends_above ? __builtin_ctzll(ends_above) : 64;
    const bool is_short = valid && seg_first >= 0 && seg_end - seg_first <= kShort;
    // and long?  Then the key 64 ahead of its first position is still its own.  A segment that holds lane 0 may begin
    // up to 64 earlier, where the keys behind lane 0 say.
    const uint32_t key0 = lane_value(key, 0), far0 = lane_value(far, 0);
    const uint64_t m_not_near = ~__ballot(near == key0);
    const int back = m_not_near ? __builtin_clzll(m_not_near) : 64;          // positions of key0 right behind lane 0
    const bool long0 = m_ends ? back + __builtin_ctzll(m_ends) > 64 : back > 0 || far0 == key0;
    const uint32_t far_first = (uint32_t)__shfl((int)far, seg_first < 0 ? 0 : seg_first);
    const bool is_long = valid && (seg_first < 0 ? long0 : far_first == key);
    const uint64_t m_short = __ballot(is_short), m_long = __ballot(is_long);
    const uint64_t pieces_below = m_piece & upto;
    const int piece_first = pieces_below ? 63 - __builtin_clzll(pieces_below) : -1;
    auto in_chunk = [&](int l) { return l > kShort && l <= kShort + kChunk; };
    const bool short_mine = is_short && in_chunk(seg_first);
    {
        // zeros at the positions of its chunk that will hold no value of this kernel's, but for those of short segments
        // that begin before it, and at those of its short segments behind the chunk
        const bool owned = q >= 0 && q < n && (in_chunk(lane) ? !is_short || short_mine : lane > kShort + kChunk && short_mine);
        // the first piece of a long id's run is the whole run if a run starts where the next piece does
        const uint64_t pieces_above = (m_piece | ~m_valid) & ~upto, runs_or_end = m_head | ~m_valid;
        const bool cut_run = is_long && !(pieces_above && ((runs_or_end >> __builtin_ctzll(pieces_above)) & 1));
        if (owned && (!((m_head >> lane) & 1) || cut_run)) contrib[(int64_t)cb * n + val] = 0.f;
        if (owned && (!((m_seg >> lane) & 1) || is_long) && !accumulate) bigpart[(int64_t)cb * n + val] = 0.f;
        if (lane == 0 && i0 > 0 && i0 >> part_bits << part_bits == i0) arrived[(i0 >> part_bits) * ((D + kColBlock - 1) / kColBlock) + cb] = 0u;
    }
    // the rows of this wave: short segments and pieces of long ones that begin in the chunk.  Taken in stretches of
    // neighbouring rows (a medium segment may lie between two).
    const uint64_t next_starts_run = (m_head | ~m_valid) >> 1, next_starts_seg = (m_seg | ~m_valid) >> 1;
    const uint64_t next_starts_piece = (m_piece | ~m_valid) >> 1, runs_below = m_head & upto;
    RowEnds ends;
    ends.park = m_long & next_starts_piece;
    ends.close = (m_short & next_starts_run) | ends.park;
    ends.id = m_short & next_starts_seg;
    const int run_first = runs_below ? 63 - __builtin_clzll(runs_below) : -1;
    // a long id's piece is a whole run if it begins at the run's head and ends where the next run starts
    ends.whole = (m_short & next_starts_run) | (ends.park & next_starts_run & __ballot(piece_first >= 0 && piece_first == run_first));
    ends.head_pos = (uint32_t)__shfl((int)val, max(is_long ? piece_first : run_first, 0));
    ends.id_pos = (uint32_t)__shfl((int)val, max(seg_first, 0));
    for (uint64_t todo = __ballot(short_mine || (is_long && in_chunk(piece_first))); todo;) {
        const int l = __builtin_ctzll(todo), e = l + __builtin_ctzll(~(todo >> l));   // rows l .. e-1
        todo &= ~(((uint64_t)1 << e) - 1);
        stream_rows<T, kVec>(g, w, runsum, contrib, bigpart, n, D, accumulate, cb, lane, key, val, l, e, ends);
    }
    }   // chunks
}

// Kernel B: the rows of w' of the ids with more than 64 positions, the shares of s[b] of their runs of several pieces,
// and the squared norms of the rows, one column block at a time.
//
// An id's positions are cut into parts at the multiples of `part` that have kSumSpan of its positions on either side, and
// every part is a workgroup's (the one whose span of kSumSpan positions holds the part's first; at most one part begins
// in a span).  The workgroup's waves take a quarter of the part's positions each, list the pieces among them and add
// their parked sums in order, eight rows in flight.  A run may be cut anywhere, so what is added up is held in three
// sums: `open` of a run that began before and ends here, `closed` of all runs that begin and end here (each squared
// at its end), and `rest` of a run that has not ended; neighbours combine by finishing the run between them.
// Waves combine through LDS.  The parts of an id leave their three sums in three rows of the workspace that they have
// read, and the last workgroup to arrive adds them up in the same way, in order: results do not depend on who is last.
// They cross between XCDs as in the one-launch reduction of the LayerNorm gradients: device-scope stores, acknowledged
// before the workgroup counts itself as arrived, and device-scope loads.
//
// Bound by latency: some 1 us each for the span, the part's positions and the combination, 2 for sixteen rows, and, for an
// id of several parts, another 5 for the arrival and the parts' sums.  Whole calls, us, a launch for the runs and one for
// the ids / one workgroup for all of an id's pieces / this: one id, bf16 B=64 T=2048 D=1024 278 / 273 / 187, presorted
// B=69 T=4815 D=26 613 / 2425 / 412; half of every example one id, bf16 B=128 T=2048 D=768 471 / 482 / 364, fp32 B=16 T=2048
// D=501 196 / 279 / 130; Zipf ids, presorted, bf16 B=16 T=2048 D=2048 128 / 125 / 124.
constexpr int kSumWaves = 4, kSumSpan = 64;
constexpr int kSumWindows = 4;                                   // windows of 64 positions that a wave lists at a time
constexpr uint32_t kNoEmit = 0xffffffffu, kEndsRun = 0x80000000u, kBeginsRun = 0x80000000u;
constexpr int kDeviceScope = 16;                                 // sc1
static_assert(kPiece == 32, "two pieces to a window");

// (Positions are 32-bit here, and what need not be unrolled is not: a workgroup runs through the code once or twice, and
// fetching the instructions is a good part of its time.)
__global__ __launch_bounds__(64 * kSumWaves, 4) void emb_sums_kernel(
    const uint32_t *keys, const uint32_t *vals, float *w, float *runsum, float *contrib, float *bigpart, uint32_t *arrived,
    uint32_t n, int part_bits, uint32_t Tn, int D, int V, int accumulate, int fill_begin, int fill_each, int sum_blocks, int fill_blocks)
{
    constexpr int kBatch = 8;                                    // rows in flight
    constexpr int kOwn = kColBlock / (64 * kSumWaves);           // columns per thread where the waves combine
    __shared__ __align__(16) uint32_t mem[kSumWaves][3 * kColBlock];           // a wave's list, then its sums: closed, open, rest
    static_assert(64 * kSumWindows + 1 <= kColBlock && 2 * 64 * 3 <= kColBlock, "the list lies where `closed` will");
    __shared__ uint32_t flags[kSumWaves], wave_emit[kSumWaves];  // opens, and ended << 1; emit_open
    __shared__ float squares[kSumWaves][kSumWaves + 1];
    __shared__ uint32_t last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncb = (D + kColBlock - 1) / kColBlock;
    if ((int)blockIdx.x >= sum_blocks) {
        fill_absent_rows(keys, n, w, fill_begin, V, D, fill_each, ((int)blockIdx.x - sum_blocks) * kSumWaves + wave, fill_blocks * kSumWaves, lane);
        return;
    }
    const int span = (int)blockIdx.x / ncb, cb = (int)blockIdx.x - span * ncb, col0 = cb * kColBlock;
    const uint32_t part = 1u << part_bits, q0 = (uint32_t)span * kSumSpan, next = ((q0 >> part_bits) + 1) << part_bits;
    // what the span and the multiples of `part` around it hold, in one trip to memory; the same in every wave
    auto key_at = [&](uint32_t q) { return q < n ? keys[q] : 0xffffffffu; };     // (also of what lies before the first: it wraps)
    const uint32_t key = key_at(q0 + lane), before = key_at(q0 + lane - 1), beyond = key_at(q0 + lane + 64), below = key_at(q0 - kSumSpan);
    const uint32_t below1 = key_at(next - kSumSpan), above1 = key_at(next + kSumSpan);
    const uint32_t below2 = key_at(next + part - kSumSpan), above2 = key_at(next + part + kSumSpan);
    const uint32_t ahead = key_at(q0 + 64 + lane * 64);
    const uint64_t starts = __ballot(key < (uint32_t)V && key != before && beyond == key);
    const uint32_t first = lane_value(key, 0);
    // the part begins at a cut (an id that is cut at q0 covers the span)
    const bool cut_lo = (q0 & (part - 1)) == 0 && first < (uint32_t)V && below == first && lane_value(beyond, 0) == first;
    if (!starts && !cut_lo) return;
    const int at_start = cut_lo ? 0 : __builtin_ctzll(starts);
    const uint32_t lo = q0 + at_start, v = lane_value(key, at_start);
    // The part's end: the next cut.  Where the next multiple of `part` is none the id begins less than kSumSpan before it
    // (and the one behind may be a cut) or ends within kSumSpan behind it.  A window at a time the keys ahead say more.
    const bool cut1 = below1 == v && above1 == v, cut2 = !cut1 && below2 == v && above2 == v, cut_hi = cut1 || cut2;
    const uint32_t limit = min((lo + kSumSpan > next ? next + part : next) + kSumSpan, n);
    const uint64_t m_ahead = ~__ballot(ahead == v);
    const uint32_t seen = m_ahead ? q0 + 64 + __builtin_ctzll(m_ahead) * 64 : limit;
    const uint32_t hi = cut1 ? next : cut2 ? next + part : min(limit, seen);             // (or before: where the id ends)

    float sub[8], closed[8];                                     // the run in hand; the wave's closed runs (its `open` goes to LDS at once)
    uint32_t opens = 0, ended = 0, emit_open = kNoEmit;          // the wave begins inside a run; a run has ended; where that run's square goes
    // What to add up: of a part, the pieces' rows of runsum and whether a run begins there (a run ends where the next one
    // begins: one more entry says so of the last); of the parts' sums, row and whether a run ends, and where its square goes.
    uint32_t *const list = mem[wave];
    const int row_bytes = min(kColBlock, D - col0) * (int)sizeof(float);
    const bool strided = D % 8 != 0;                             // (runsum is 256-byte aligned)
    auto column = [&](int j) { return strided ? j * 64 + lane : lane * 8 + j; };
    // Adds up the rows of the list.  Eight neighbouring columns per lane, or columns 64 apart (any D).  shared: rows that
    // other workgroups of this launch have stored.
    auto add_list = [&](int count, bool shared) {
        for (int k = 0; k < count; k += kBatch) {
            const int at = min(k + lane % kBatch, count - 1);
            uint32_t rows, emits;                                // row, and kEndsRun; where the square of a run of several goes
            if (shared) {
                rows = list[2 * at];
                emits = list[2 * at + 1];
            } else {
                const uint32_t here = list[at], after = list[at + 1];
                rows = (here & ~kBeginsRun) | (after & kBeginsRun ? kEndsRun : 0u);
                emits = after & ~here & kBeginsRun ? here : kNoEmit;
            }
            int at_lane = lane * (strided ? 4 : 32), open_row = -1;
            asm volatile("" : "+v"(at_lane));                    // (the constants behind it go into the instructions, not into registers)
            float add[kBatch][8], sq[kBatch];                    // all loads first, then the additions in order
            auto buffer = [&](int u) {                           // a row as a buffer: columns behind its end read as zeros
                return make_rsrc(runsum + (int64_t)(lane_value(rows, u) & ~kEndsRun) * D + col0, row_bytes);
            };
            auto eight = [&](auto aux) {
                constexpr int kAux = decltype(aux)::value;
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const rsrc_t r = buffer(u);
                    unpack_row8(Row8<float>{__builtin_bit_cast(float4, buffer_load16<kAux>(r, at_lane)), __builtin_bit_cast(float4, buffer_load16<kAux>(r, at_lane + 16))}, add[u]);
                }
            };
            if (strided) {
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const rsrc_t r = buffer(u);
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        add[u][j] = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, at_lane + j * 256, 0, kDeviceScope));
                }
            } else if (shared) {
                eight(std::integral_constant<int, kDeviceScope>{});
            } else {
                eight(std::integral_constant<int, 0>{});
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                sq[u] = 0.f;
                if (k + u >= count) continue;
#pragma unroll
                for (int j = 0; j < 8; ++j) sub[j] += add[u][j];
                if (!(lane_value(rows, u) & kEndsRun)) continue;
                if (opens && !ended) {
                    emit_open = lane_value(emits, u);
                    open_row = u;
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        list[kColBlock + column(j)] = __builtin_bit_cast(uint32_t, sub[j]);
                        sub[j] = 0.f;
                    }
                }
                ended = 1;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    sq[u] = fmaf(sub[j], sub[j], sq[u]);
                    closed[j] += sub[j];
                    sub[j] = 0.f;
                }
            }
            const bool mine = lane < kBatch && k + lane < count && emits != kNoEmit && lane != open_row;
            if (__any(mine)) {
                const float total = wave_sums8(sq, lane);
                if (mine) contrib[(int64_t)cb * n + emits] = total;
            }
        }
    };
    auto own_lds = [&]() {                                       // a wave's own LDS accesses, by other lanes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    double tot_open[kOwn], tot_closed[kOwn], tot_rest[kOwn];     // the workgroup's sums of columns tid, tid + 256, ...
    auto combine = [&]() {
        __syncthreads();                                         // the lists have been read
        if (strided) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                list[j * 64 + lane] = __builtin_bit_cast(uint32_t, closed[j]);
                list[2 * kColBlock + j * 64 + lane] = __builtin_bit_cast(uint32_t, sub[j]);
            }
        } else {
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                *reinterpret_cast<u32x4_t *>(list + lane * 8 + h) = __builtin_bit_cast(u32x4_t, make_float4(closed[h], closed[h + 1], closed[h + 2], closed[h + 3]));
                *reinterpret_cast<u32x4_t *>(list + 2 * kColBlock + lane * 8 + h) = __builtin_bit_cast(u32x4_t, make_float4(sub[h], sub[h + 1], sub[h + 2], sub[h + 3]));
            }
        }
        if (lane == 0) {
            flags[wave] = opens | ended << 1;
            wave_emit[wave] = emit_open;
        }
        __syncthreads();
        uint32_t fl[kSumWaves], m[kSumWaves][kOwn], a[kSumWaves][kOwn], z[kSumWaves][kOwn];
#pragma unroll
        for (int u = 0; u < kSumWaves; ++u) {
            fl[u] = (uint32_t)__builtin_amdgcn_readfirstlane((int)flags[u]);
#pragma unroll
            for (int o = 0; o < kOwn; ++o) {
                const int c = tid + o * 64 * kSumWaves;
                m[u][o] = mem[u][c];
                a[u][o] = mem[u][kColBlock + c];
                z[u][o] = mem[u][2 * kColBlock + c];
            }
        }
#pragma unroll
        for (int o = 0; o < kOwn; ++o) tot_open[o] = tot_closed[o] = tot_rest[o] = 0.0;
        bool any = false;
        uint32_t to_emit = 0;                                    // waves whose first end completes a run of the part
#pragma unroll
        for (int u = 0; u < kSumWaves; ++u) {
            const bool u_opens = fl[u] & 1, u_ends = fl[u] & 2;
            const bool before_part = !any && (fl[0] & 1);        // that run began before the part
            float sq = 0.f;
#pragma unroll
            for (int o = 0; o < kOwn; ++o) {
                const double rest = (double)__builtin_bit_cast(float, z[u][o]), r = tot_rest[o] + (double)__builtin_bit_cast(float, a[u][o]);
                if (u_ends) {
                    tot_closed[o] += (double)__builtin_bit_cast(float, m[u][o]);
                    if (u_opens && before_part) tot_open[o] = r;
                    if (u_opens && !before_part) {
                        tot_closed[o] += r;
                        sq = fmaf((float)r, (float)r, sq);
                    }
                    tot_rest[o] = rest;
                } else {
                    tot_rest[o] += rest;
                }
            }
            if (u_ends && u_opens && !before_part) {
                to_emit |= 1u << u;
                sq = wave_sum(sq);
                if (lane == 0) squares[u][wave] = sq;
            }
            any = any || u_ends;
        }
        if (!to_emit) return;
        __syncthreads();
        if (tid < kSumWaves && ((to_emit >> tid) & 1)) {
            float t = 0.f;
            for (int u = 0; u < kSumWaves; ++u) t += squares[tid][u];
            contrib[(int64_t)cb * n + wave_emit[tid]] = t;
        }
    };

    // ---- first the rows of the part, then, for the last workgroup of several, the sums that the parts have left
    uint32_t first_cut = 0, parts = 1;
    uint32_t park[3] = {0, 0, 0};                                // rows of runsum for the part's three sums
#pragma unroll 1
    for (bool over_parts = false;; over_parts = true) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sub[j] = closed[j] = 0.f;
        ended = opens = 0;
        emit_open = kNoEmit;
        // a wave takes a quarter of the windows of 64 positions, or of the parts
        const uint32_t it_first = over_parts ? 0 : lo / 64, its = over_parts ? parts : (hi - 1) / 64 - it_first + 1;
        const uint32_t per = (its + kSumWaves - 1) / kSumWaves, it_begin = it_first + min(wave * per, its);
        const uint32_t it_end = min(it_begin + per, it_first + its);
        // the example of the position before the windows in hand if it is the id's, and the next windows' pairs, on their
        // way while rows are added
        uint32_t ex_before = kNoEmit, next_key[kSumWindows], next_val[kSumWindows], key_behind = 0, val_behind = 0;
        auto fetch = [&](uint32_t window) {
#pragma unroll
            for (int x = 0; x < kSumWindows; ++x) {
                const uint32_t q = (window + x) * 64 + lane;
                next_key[x] = key_at(q);
                next_val[x] = q < n ? vals[q] : 0u;
            }
            const uint32_t q = (window + kSumWindows) * 64;
            key_behind = key_at(q);
            val_behind = q < n ? vals[q] : 0u;
        };
        if (!over_parts && it_begin < it_end) {
            const uint32_t q = it_begin * 64 - 1, key_before = key_at(q), val_before = q < n ? vals[q] : 0u;
            fetch(it_begin);
            if (key_before == v) ex_before = val_before / Tn;
        }
        if (!over_parts && (cut_lo || cut_hi)) {
            // the id's cuts are the multiples first_cut .. last_cut of `part` (found while the windows are on their way)
            const uint32_t some = (cut_lo ? lo : hi) >> part_bits, most = n >> part_bits;
            const bool up = lane >= 32;
            const uint32_t found = half_wave_first_not(up ? some : 1, up ? most - some + 1 : some - 1, lane, [&](uint32_t k) {
                return up ? key_at((k << part_bits) + kSumSpan) <= v : key_at((k << part_bits) - kSumSpan) < v;
            });
            first_cut = lane_value(found, 0);
            const uint32_t last_cut = lane_value(found, 32) - 1;
            parts = last_cut - first_cut + 2;
            // the sums go to the rows of the last three positions before the part's end, or, of the id's last part, of the first three
            const uint32_t base = cut_hi ? hi - 3 : lo;
#pragma unroll
            for (int i = 0; i < 3; ++i) park[i] = vals[base + i];
        }
#pragma unroll 1
        for (uint32_t it = it_begin; it < it_end; it += over_parts ? 64 : kSumWindows) {
            int count = 0;
            own_lds();
            if (!over_parts) {
                uint32_t ex[kSumWindows + 1], val[kSumWindows];  // the examples of the id's positions, kNoEmit elsewhere
#pragma unroll
                for (int x = 0; x < kSumWindows; ++x) {
                    val[x] = next_val[x];
                    ex[x] = next_key[x] == v ? val[x] / Tn : kNoEmit;
                }
                ex[kSumWindows] = key_behind == v ? val_behind / Tn : kNoEmit;
                if (it + kSumWindows < it_end) fetch(it + kSumWindows);
                bool goes_on = false;                            // the last run listed, behind the last position
#pragma unroll
                for (int x = 0; x < kSumWindows; ++x) {
                    const uint32_t q = (it + x) * 64 + lane;
                    const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp((int)ex_before, (int)ex[x], 0x138, 0xf, 0xf, false);   // wave_shr:1
                    const bool mine = ex[x] != kNoEmit && q >= lo && q < hi && it + x < it_end, begins = ex[x] != prev;
                    const bool piece = mine && (begins || lane % kPiece == 0);                   // (windows begin at multiples of kPiece)
                    const uint64_t m_mine = __ballot(mine), m_new = __ballot(begins), m_piece = __ballot(piece);
                    ex_before = lane_value(ex[x], 63);
                    if (!m_mine) continue;
                    if (it == it_begin && x == 0) opens = (m_new >> __builtin_ctzll(m_mine)) & 1 ? 0 : 1;
                    if (piece) {
                        const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(m_piece >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m_piece, (uint32_t)count));
                        list[to] = val[x] | (begins ? kBeginsRun : 0u);
                    }
                    count += __builtin_popcountll(m_piece);
                    const uint64_t behind = m_new & ~m_mine;     // the id's positions are neighbours
                    goes_on = m_mine >> 63 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)ex[x + 1]) == ex_before
                                           : !((behind >> (64 - __builtin_clzll(m_mine))) & 1);
                }
                if (lane == 0) list[count] = goes_on ? 0u : kBeginsRun;
            } else {                                             // part m lies between cuts first_cut + m - 1 and first_cut + m
                const uint32_t m = it + lane;
                const bool in = m < it_end, has_lo = in && m > 0, has_hi = in && m < parts - 1;
                const uint32_t at_lo = (first_cut + m - 1) << part_bits, at_hi = at_lo + part, at = has_hi ? at_hi - 3 : at_lo;
                auto position = [&](bool there, uint32_t q) { return there ? vals[q] : 0u; };
                const uint32_t r0 = position(in, at), r1 = position(in, at + 1), r2 = position(in, at + 2);
                const uint32_t p_lo = position(has_lo, at_lo), e_before = position(has_lo, at_lo - 1) / Tn;
                const uint32_t e_last = position(has_hi, at_hi - 1) / Tn, e_behind = position(has_hi, at_hi) / Tn;
                const bool from = has_lo && p_lo / Tn == e_before, on = has_hi && e_last == e_behind;   // a run goes on over the lower cut, over the upper
                const bool through = from && on && p_lo / Tn == e_last;
                const uint64_t m_open = __ballot(from && !through), m_closed = __ballot(in && !through), m_rest = __ballot(on);
                const uint64_t lower = ((uint64_t)1 << lane) - 1;
                int to = __builtin_popcountll(m_open & lower) + __builtin_popcountll(m_closed & lower) + __builtin_popcountll(m_rest & lower);
                if (it == it_begin) opens = (uint32_t)(__ballot(from) & 1);
                if (from && !through) {
                    list[2 * to] = r0 | kEndsRun;
                    list[2 * to++ + 1] = p_lo;
                }
                if (in && !through) {
                    list[2 * to] = r1 | kEndsRun;
                    list[2 * to++ + 1] = kNoEmit;
                }
                if (on) {
                    list[2 * to] = r2;
                    list[2 * to + 1] = kNoEmit;
                }
                count = __builtin_popcountll(m_open) + __builtin_popcountll(m_closed) + __builtin_popcountll(m_rest);
            }
            own_lds();
            add_list(count, over_parts);
        }
        combine();
        if (over_parts || (!cut_lo && !cut_hi)) break;
        // one of several parts
#pragma unroll
        for (int o = 0; o < kOwn; ++o) {
            const int col = col0 + tid + o * 64 * kSumWaves;
            if (col < D) {
                __hip_atomic_store(runsum + (int64_t)park[0] * D + col, (float)tot_open[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(runsum + (int64_t)park[1] * D + col, (float)tot_closed[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(runsum + (int64_t)park[2] * D + col, (float)tot_rest[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        // every thread: this thread's sums have reached the memory that all XCDs share
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
            last = __hip_atomic_fetch_add(arrived + (int64_t)first_cut * ncb + cb, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
        __syncthreads();
        if (!last) return;
    }
    // ---- the id's row of w' is complete
    float sq = 0.f;
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
        const int col = col0 + tid + o * 64 * kSumWaves;
        if (col < D) {
            float *p = w + (int64_t)v * D + col;
            const float sum = (float)(tot_closed[o] + (accumulate ? (double)*p : 0.0));
            __builtin_nontemporal_store(sum, p);
            sq = fmaf(sum, sum, sq);
        }
    }
    if (accumulate) return;
    sq = wave_sum(sq);
    if (lane == 0) squares[wave][kSumWaves] = sq;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
        for (int u = 0; u < kSumWaves; ++u) t += squares[u][kSumWaves];
        bigpart[(int64_t)cb * n + vals[parts > 1 ? first_cut << part_bits : lo]] = t;
    }
}

// partial sums of squares of w (accumulate mode: every row counts, not only those touched).  Four 16-byte
// loads in flight per thread; every thread's own order of additions is fixed.
__global__ __launch_bounds__(256) void emb_wnorm_kernel(const float *w, int64_t n, double *part)
{
    __shared__ double slots[4];
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double t = 0.0;
    if ((reinterpret_cast<uintptr_t>(w) & 15u) == 0) {
        const float4 *w4 = reinterpret_cast<const float4 *>(w);
        const int64_t n4 = n / 4;
        double t1 = 0.0, t2 = 0.0, t3 = 0.0;
        auto sq4 = [](const float4 &v) {
            return (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
        };
        for (; i + 3 * stride < n4; i += 4 * stride) {
            const float4 a = w4[i], b = w4[i + stride], c = w4[i + 2 * stride], d = w4[i + 3 * stride];
            t += sq4(a); t1 += sq4(b); t2 += sq4(c); t3 += sq4(d);
        }
        for (; i < n4; i += stride) t += sq4(w4[i]);
        t = (t + t1) + (t2 + t3);
        i = n4 * 4 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    }
    for (; i < n; i += stride) t += (double)w[i] * (double)w[i];
    t = block_sum_f64(t, slots);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// s[b] = sum over column blocks and positions of example b of contrib; big_sq from its parts.  fp64, fixed order.
__global__ __launch_bounds__(1024) void emb_final_kernel(const float *contrib, const float *bigpart,
                                                         const double *wpart, int nwpart, float *s, float *big_sq,
                                                         int B, int Tn, int ncb, int64_t n)
{
    __shared__ double slots[16];
    const int b = blockIdx.x;
    double t = 0.0;
    if (b < B) {
        for (int c = 0; c < ncb; ++c)
            for (int i = threadIdx.x; i < Tn; i += 1024) t += (double)contrib[(int64_t)c * n + (int64_t)b * Tn + i];
        t = block_sum_f64(t, slots);
        if (threadIdx.x == 0) s[b] = (float)t;
    } else if (big_sq) {
        if (wpart) {
            for (int i = threadIdx.x; i < nwpart; i += 1024) t += wpart[i];
        } else {
            // sixteen 16-byte loads in flight per thread; every thread's order of additions is fixed
            double part[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) part[u] = 0.0;
            const int64_t m = (int64_t)ncb * n, m4 = m / 4;       // bigpart is 256-byte aligned
            const float4 *big4 = reinterpret_cast<const float4 *>(bigpart);
            auto sum4 = [](const float4 &q) { return ((double)q.x + (double)q.y) + ((double)q.z + (double)q.w); };
            int64_t i = threadIdx.x;
            for (; i + 15 * 1024 < m4; i += 16 * 1024) {
                float4 q[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) q[u] = big4[i + u * 1024];
#pragma unroll
                for (int u = 0; u < 16; ++u) part[u] += sum4(q[u]);
            }
            for (; i < m4; i += 1024) part[0] += sum4(big4[i]);
            for (i = m4 * 4 + threadIdx.x; i < m; i += 1024) part[1] += (double)bigpart[i];
#pragma unroll
            for (int u = 0; u < 16; ++u) t += part[u];
        }
        t = block_sum_f64(t, slots);
        if (threadIdx.x == 0) big_sq[0] = (float)t;
    }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }


int key_bits(int V)
{
    int bits = 1;
    while (bits < 32 && ((uint64_t)1 << bits) <= (uint64_t)V) ++bits;   // keys run up to V inclusive
    return bits;
}

struct EmbPlan {
    int64_t n;
    int ncb, ntiles;
    bool own_sort;          // few enough positions for the library's own sort
    size_t off_keys_in, off_keys_out, off_vals_in, off_vals_out, off_contrib, off_bigpart, off_wpart, off_tiles, off_temp, off_runsum;
    size_t temp_bytes, bytes;
};

bool emb_shape_ok(int B, int T, int D, int V)
{
    return B > 0 && T > 0 && D > 0 && V > 0 && (int64_t)B * T < ((int64_t)1 << 31) && V < (1 << 30);
}

// radix: whether rocPRIM's sort will run (its temporary storage is sized by that library for the current device, which
// takes longer than a launch: not asked for where our own sort is used).
hipError_t make_emb_plan(int B, int T, int D, int V, bool radix, EmbPlan &p)
{
    p.n = (int64_t)B * T;
    p.ncb = (D + kColBlock - 1) / kColBlock;
    const int64_t ntiles = (p.n + kSortTile - 1) / kSortTile;
    p.own_sort = ntiles <= kSortTiles;
    p.ntiles = (int)ntiles;
    size_t temp = 0;
    if (radix) {
        const hipError_t e = rocprim::radix_sort_pairs(nullptr, temp, (const uint32_t *)nullptr, (uint32_t *)nullptr,
                                                       (const uint32_t *)nullptr, (uint32_t *)nullptr, (size_t)p.n, 0,
                                                       key_bits(V), (hipStream_t)0);
        if (e != hipSuccess) return e;
    }
    const size_t arr = align256((size_t)p.n * sizeof(uint32_t)), f = align256((size_t)p.ncb * p.n * sizeof(float));
    const size_t in = p.own_sort ? 0 : arr;       // what rocPRIM's sort reads
    p.off_keys_in = 0;
    p.off_keys_out = p.off_keys_in + in;
    p.off_vals_in = p.off_keys_out + arr;
    p.off_vals_out = p.off_vals_in + in;
    p.off_contrib = p.off_vals_out + arr;
    p.off_bigpart = p.off_contrib + f;
    p.off_wpart = p.off_bigpart + f;
    p.off_tiles = p.off_wpart + align256(kNormBlocks * sizeof(double));
    p.off_temp = p.off_tiles + (p.own_sort ? align256((size_t)ntiles * kSortTile * sizeof(uint64_t)) : 0);
    p.temp_bytes = temp;
    p.off_runsum = p.off_temp + align256(temp);
    p.bytes = p.off_runsum + align256((size_t)p.n * D * sizeof(float));
    return hipSuccess;
}

// The library's own sort of the ids into (sorted_ids, sorted_pos): two launches.
template <typename W>
hipError_t own_sort(const void *ids, int ids_are_int64, const EmbPlan &p, int V, void *tiles, uint32_t *sorted_ids,
                    uint32_t *sorted_pos, const ShadowFill &fill, hipStream_t st)
{
    W *t = static_cast<W *>(tiles);
    hipError_t e = launch(emb_tile_sort_kernel<W>, dim3(p.ntiles), dim3(kSortThreads), 0, st, ids, ids_are_int64, p.n, V, t);
    if (e != hipSuccess) return e;
    return launch(emb_rank_kernel<W>, dim3(p.ntiles * (kSortTile / kRankThreads) + fill.blocks), dim3(kRankThreads),
                  (size_t)p.ntiles * kSamples * sizeof(W), st, t, p.ntiles, p.n, sorted_ids, sorted_pos, fill);
}

hipError_t sort_ids(const void *ids, int ids_are_int64, const EmbPlan &p, int V, char *ws, uint32_t *sorted_ids,
                    uint32_t *sorted_pos, const ShadowFill &fill, hipStream_t st)
{
    if (p.own_sort)
        return sort_words_are_32(V) ? own_sort<uint32_t>(ids, ids_are_int64, p, V, ws + p.off_tiles, sorted_ids, sorted_pos, fill, st)
                                    : own_sort<uint64_t>(ids, ids_are_int64, p, V, ws + p.off_tiles, sorted_ids, sorted_pos, fill, st);
    uint32_t *keys_in = reinterpret_cast<uint32_t *>(ws + p.off_keys_in), *vals_in = reinterpret_cast<uint32_t *>(ws + p.off_vals_in);
    const hipError_t e = launch(emb_prepare_kernel, dim3((unsigned)((p.n + 255) / 256)), dim3(256), 0, st, ids, ids_are_int64,
                                keys_in, vals_in, p.n, V);
    if (e != hipSuccess) return e;
    size_t temp = p.temp_bytes;
    return rocprim::radix_sort_pairs(ws + p.off_temp, temp, keys_in, sorted_ids, vals_in, sorted_pos, (size_t)p.n, 0,
                                     key_bits(V), st);
}

}  // namespace
}  // namespace lnpegn

using namespace lnpegn;

extern "C" {

size_t embedding_pegn_workspace_bytes(int B, int T, int D, int V)
{
    if (!emb_shape_ok(B, T, D, V)) return 0;
    EmbPlan p;
    return make_emb_plan(B, T, D, V, true, p) == hipSuccess ? p.bytes : 0;
}

// The call behind embedding_pegn (ids: sorted here) and embedding_pegn_presorted (sorted_ids / sorted_pos: by the
// caller, with embedding_sort_ids).
static int run_embedding(const void *ids, int ids_are_int64, const uint32_t *sorted_ids, const uint32_t *sorted_pos,
                         const void *g, float *w, float *s, float *big_sq, int B, int T, int D, int V, lnpegn_dtype dt,
                         void *workspace, size_t workspace_bytes, unsigned flags, void *stream)
{
    if (!emb_shape_ok(B, T, D, V) || !g || !w || !s || !workspace) return LNPEGN_EINVAL;
    if (!ids && (!sorted_ids || !sorted_pos)) return LNPEGN_EINVAL;
    if (flags & ~(unsigned)LNPEGN_ACCUMULATE) return LNPEGN_EINVAL;
    if (dt != LNPEGN_F32 && dt != LNPEGN_BF16) return LNPEGN_EUNSUPPORTED;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return LNPEGN_EINVAL;
    EmbPlan p;
    const bool radix = ids && (int64_t)B * T > (int64_t)kSortTiles * kSortTile;
    if (make_emb_plan(B, T, D, V, radix, p) != hipSuccess) return LNPEGN_EHIP;
    if (workspace_bytes < p.bytes) return LNPEGN_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int accumulate = (flags & LNPEGN_ACCUMULATE) ? 1 : 0;
    char *ws = static_cast<char *>(workspace);
    const uint32_t *keys = ids ? reinterpret_cast<uint32_t *>(ws + p.off_keys_out) : sorted_ids;
    const uint32_t *vals = ids ? reinterpret_cast<uint32_t *>(ws + p.off_vals_out) : sorted_pos;
    float *contrib = reinterpret_cast<float *>(ws + p.off_contrib);
    float *bigpart = reinterpret_cast<float *>(ws + p.off_bigpart);
    double *wpart = reinterpret_cast<double *>(ws + p.off_wpart);
    float *runsum = reinterpret_cast<float *>(ws + p.off_runsum);
    // 1. the ids sorted, and beside the library's own sort the first rows of w' cleared: whole rows that end on the boundary
    // of a line, or all of a w' that is no more than that.
    const int esz = dt == LNPEGN_BF16 ? 2 : 4;
    const int64_t row_bytes = (int64_t)D * 4;
    // rows that are whole lines of 128 bytes, where 64 KB are enough for that
    const int lines = 32 / (int)((D & -D) < 32 ? (D & -D) : 32), whole = lines * row_bytes <= 2 * kFillMost ? lines : 1;
    const int64_t w_mib = V * row_bytes >> 20;
    // Only where there is more of it than the kernels behind the sort hide, or so few positions that they hide nothing.  us a call,
    // without / with: fp32 V=50257 D=488 (94 MiB) n=4096 40.2 / 39.1, V=37197 D=840 (119) n=4096 46.3 / 44.1; bf16 V=50257 D=448 (86) n=8192
    // 44.0 / 45.3, D=512 (98) n=1024 36.8 / 37.4, D=768 (147) n=8192 50.9 / 49.8, D=640 (123) n=4096 40.6 / 40.3 but n=32768 62.9 / 64.1; V=32000
    // D=512 (62) n=256 31.9 / 29.3, n=1024 33.4 / 32.9, n=4096 36.4 / 36.9, V=8000 D=768 (23) n=256 27.8 / 26.0, n=4096 35.6 / 35.1, n=32768 59.5 / 59.5;
    // rows that are no whole lines, V=32000 D=1693 n=1024 84.1 / 79.9, n=16384 126.1 / 126.5.
    const bool much = w_mib >= (esz == 4 ? 90 : p.n > 16384 ? 144 : 108) && (lines <= 4 || p.n <= 4096);
    const bool few = p.n <= (w_mib < 32 ? 4096 : w_mib < 64 ? 1024 : 256);
    int cleared = 0;                                              // rows
    if (ids && p.own_sort && !accumulate && (reinterpret_cast<uintptr_t>(w) & 15u) == 0 && p.n * esz < (int64_t)V * 4 && (much || few)) {
        const int64_t rows = kShadowMost / row_bytes;
        cleared = rows < V ? (int)(rows / lines * lines) : V;     // (nor less than 16 bytes)
    }
    const ShadowFill shadow{w, (int64_t)cleared * D, (int)(((int64_t)cleared * row_bytes + kShadowBytes - 1) / kShadowBytes)};
    if (ids && sort_ids(ids, ids_are_int64, p, V, ws, const_cast<uint32_t *>(keys), const_cast<uint32_t *>(vals), shadow, st) != hipSuccess)
        return LNPEGN_EHIP;
    // 2. runs, and beside them the fill of the rows no id selects
    // 8 columns per lane: 16 bytes of bf16, 32 bytes of fp32; rows must keep that alignment
    const bool vec = (reinterpret_cast<uintptr_t>(g) & 15u) == 0 && ((int64_t)D * esz) % 16 == 0 && D % 8 == 0;
    const int64_t chunks = (p.n + kChunk - 1) / kChunk;
    const int runs_x = (int)(chunks < g_emb_run_blocks ? chunks : g_emb_run_blocks), runs_y = (p.ncb + kWavesPerBlock - 1) / kWavesPerBlock;
    // The rows filled beside kernel A; the rest beside kernel B.  The shares meet on the boundary of a line: their waves take whole
    // lines, counted from where a share begins.  (us, shares that meet at any row / this: V=50257 presorted fp32 D=1512 n=1024 80.2 /
    // 74.0, sorted in the call bf16 D=1688 n=2115 91.9 / 79.8, D=1448 n=406 77.4 / 66.2.)
    // Most of it beside kernel B: 128 MiB, of a w' of which half is well above 40 MiB, the larger the fewer the positions.  us a
    // presorted call, V=50257, 40 MiB at most / 128: bf16 D=512 (98 MiB) n=4096 39.1 / 39.5, fp32 D=552 (106) n=4096 42.7 / 41.8 but n=256
    // 35.9 / 36.7, D=768 (147) n=256 42.5 / 42.3, n=8192 54.6 / 50.9, D=2048 n=256 93.3 / 91.6, n=32768 131.6 / 123.1; V=32000 fp32 D=1024 (125) n=256
    // 39.3 / 40.0, n=1024 41.2 / 40.7.  Not of rows that are whole lines only by eight and more: bf16 D=1001 (192) n=1024 87.4 / 90.8,
    // V=32000 D=1693 (207) n=16384 125.1 / 128.5.
    const int64_t late_most = (lines <= 4 && w_mib >= (p.n < 1024 ? 144 : p.n < 4096 ? 112 : 96) ? kFillLateLarge : kFillLateBytes) / row_bytes;
    const int64_t half = (V - cleared) / 2, late = half < late_most ? half : late_most;
    const int meet = (V - (int)late) / whole * whole, fill_end = meet > cleared ? meet : V - (int)late;
    const int fill_a = accumulate ? 0 : fill_end - cleared, fill_b = accumulate ? 0 : V - fill_end;
    // Rows to a wave: 8 to 32 KB, so that there are many waves and the search for their ids is hidden, and whole lines.
    auto rows_each = [&](int rows) {
        int64_t bytes = rows * row_bytes / kFillBlocks;
        bytes = bytes < kFillLeast ? kFillLeast : bytes > kFillMost ? kFillMost : bytes;
        int64_t each = bytes / row_bytes > 1 ? bytes / row_bytes : 1;
        each = (each + whole - 1) / whole * whole;
        return (int)(each < 64 ? each : 64);
    };
    auto blocks_for = [&](int rows, int each) {
        const int64_t most = ((int64_t)rows + each * kWavesPerBlock - 1) / (each * kWavesPerBlock);
        return (int)(most < kFillBlocks ? most : kFillBlocks);
    };
    const int each_a = rows_each(fill_a), each_b = rows_each(fill_b);
    const int fill_blocks = blocks_for(fill_a, each_a), fill_blocks_b = blocks_for(fill_b, each_b), medium_blocks = (int)chunks * runs_y;
    hipError_t runs_status = hipSuccess;
    // kernel B's counters lie where the sort had its words; parts large enough that they fit
    const size_t counter_bytes = p.own_sort ? p.off_temp - p.off_tiles : p.off_keys_out - p.off_keys_in;
    uint32_t *arrived = reinterpret_cast<uint32_t *>(ws + (p.own_sort ? p.off_tiles : p.off_keys_in));
    // Parts small enough to run side by side, large enough that few sums are left to add; small batches are spared the
    // second level.  Parts of 1024 / 2048 / 4096 positions, us: Zipf ids in 8192 47.3 / 48.3 / 44.8 (D=768), in 32768
    // 36.6 / 39.0 / 43.9 (D=512, V=256); one id in 32768 67.6 / 70.2 / 76.7 (D=768), in 131072 164 / 150 / 149; half of
    // 262144 one id 295 / 273 / 266; one id in 306557 415 / 387 / 380.
    int part_bits = p.n <= 16384 ? 12 : p.n <= 65536 ? 10 : p.n <= 131072 ? 11 : p.n <= 262144 ? 12 : 13;
    while ((size_t)((p.n >> part_bits) + 1) * p.ncb * sizeof(uint32_t) > counter_bytes && p.n >> part_bits) ++part_bits;
    auto runs = [&](auto kernel, auto *gp) {
        auto go = [&](int medium, int fill, int run) {
            return launch(kernel, dim3((unsigned)(medium + fill + run)), dim3(64 * kWavesPerBlock), 0, st, gp, keys, vals, w, runsum, contrib,
                          bigpart, arrived, p.n, part_bits, T, D, V, accumulate, medium, cleared, fill_end, each_a, fill, runs_x);
        };
        // a launch holds less than 2^32 threads: the medium segments of nearly 2^28 positions need one of their own
        const bool one = ((int64_t)medium_blocks + fill_blocks + runs_x * runs_y) * 64 * kWavesPerBlock <= 0xffffffffll;
        if (!one) runs_status = go(medium_blocks, 0, 0);
        if (runs_status == hipSuccess) runs_status = go(one ? medium_blocks : 0, fill_blocks, runs_x * runs_y);
    };
    if (dt == LNPEGN_BF16) {
        if (vec) runs(emb_runs_kernel<bf16_t, true>, static_cast<const bf16_t *>(g));
        else runs(emb_runs_kernel<bf16_t, false>, static_cast<const bf16_t *>(g));
    } else {
        if (vec) runs(emb_runs_kernel<float, true>, static_cast<const float *>(g));
        else runs(emb_runs_kernel<float, false>, static_cast<const float *>(g));
    }
    if (runs_status != hipSuccess) return LNPEGN_EHIP;
    // 3. the parked sums
    const int64_t sum_blocks = (p.n + kSumSpan - 1) / kSumSpan * p.ncb;
    if (launch(emb_sums_kernel, dim3((unsigned)(sum_blocks + fill_blocks_b)), dim3(64 * kSumWaves), 0, st, keys, vals, w, runsum, contrib, bigpart,
               arrived, (uint32_t)p.n, part_bits, (uint32_t)T, D, V, accumulate, fill_end, each_b, (int)sum_blocks, fill_blocks_b) != hipSuccess)
        return LNPEGN_EHIP;
    // 4. the norms
    const bool wnorm = accumulate && big_sq;
    if (wnorm) {
        if (launch(emb_wnorm_kernel, dim3(kNormBlocks), dim3(256), 0, st, w, (int64_t)V * D, wpart) != hipSuccess) return LNPEGN_EHIP;
    }
    return launch(emb_final_kernel, dim3(B + 1), dim3(1024), 0, st, contrib, bigpart, wnorm ? wpart : nullptr, kNormBlocks, s, big_sq, B, T,
                  p.ncb, p.n) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int embedding_pegn(const void *ids, int ids_are_int64, const void *g, float *w, float *s, float *big_sq, int B, int T,
                   int D, int V, lnpegn_dtype dt, void *workspace, size_t workspace_bytes, unsigned flags, void *stream)
{
    if (!ids) return LNPEGN_EINVAL;
    return run_embedding(ids, ids_are_int64, nullptr, nullptr, g, w, s, big_sq, B, T, D, V, dt, workspace,
                         workspace_bytes, flags, stream);
}

int embedding_sort_ids(const void *ids, int ids_are_int64, int B, int T, int V, uint32_t *sorted_ids,
                       uint32_t *sorted_pos, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!emb_shape_ok(B, T, 1, V) || !ids || !sorted_ids || !sorted_pos || !workspace) return LNPEGN_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return LNPEGN_EINVAL;
    EmbPlan p;
    if (make_emb_plan(B, T, 1, V, (int64_t)B * T > (int64_t)kSortTiles * kSortTile, p) != hipSuccess) return LNPEGN_EHIP;
    if (workspace_bytes < p.bytes) return LNPEGN_EWORKSPACE;
    return sort_ids(ids, ids_are_int64, p, V, static_cast<char *>(workspace), sorted_ids, sorted_pos, ShadowFill{},
                    static_cast<hipStream_t>(stream)) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int embedding_pegn_presorted(const uint32_t *sorted_ids, const uint32_t *sorted_pos, const void *g, float *w, float *s,
                             float *big_sq, int B, int T, int D, int V, lnpegn_dtype dt, void *workspace,
                             size_t workspace_bytes, unsigned flags, void *stream)
{
    if (!sorted_ids || !sorted_pos) return LNPEGN_EINVAL;
    return run_embedding(nullptr, 0, sorted_ids, sorted_pos, g, w, s, big_sq, B, T, D, V, dt, workspace,
                         workspace_bytes, flags, stream);
}

}  // extern "C"
