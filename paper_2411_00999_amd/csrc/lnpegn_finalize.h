// Second level of the two-level deterministic reduction: sums of the per-chunk column sums,
// the per-example squared norms (Appendix B steps 2 and 6), the batch gradients (steps 3
// and 7) and the gradient-noise-scale estimator (Section 2.1, Eq. 3-5).  Every sum runs in a
// fixed order, in fp64, so results do not depend on scheduling.  Two forms: one launch whose workgroups each
// finish a slab of columns (reduce_slab_kernel), and two levels of launches for many examples of many chunks.
#pragma once
#include "lnpegn_device.h"

namespace lnpegn {

constexpr int kTile = 256;  // columns per workgroup

struct ReduceArgs {
    const float *part;     // [n_slots][2][D] column sums per chunk
    float *grp;            // [G1][2][D] sums per group of chunks
    double *part_s;        // [n_ex][ntile][2] per-example squared norms per tile
    double *part_big;      // [ntile][2] squared norms of the batch gradients per tile
    float *dgamma;         // [D]
    float *dbeta;          // [D]
    float *pe_gamma_sq;    // [n_ex]
    float *pe_beta_sq;
    float *big_sq;         // [2] or null
    int n_slots;
    int gs;                // chunks per group (the last group may be short)
    int G1;                // number of groups
    int n_ex;              // examples whose squared norms are taken from their chunks' sums here (Appendix B
                           // steps 2, 6); 0 when there are none or the row kernel wrote them itself
    int ex_gs;             // chunks per example: example b owns chunks [b*ex_gs, (b+1)*ex_gs)
    int D;
    int ntile;
    int accumulate;        // dgamma, dbeta: add to what is there (gradient accumulation) instead of overwrite
    int nslab;             // slab kernel: slabs of columns
    double *slab;          // [n_ex + 1][nslab][2] squared norms per slab: the examples', then the batch gradients'
    unsigned *arrived;     // workgroups that have left theirs
};

// An example's chunks are also one of the groups (as many groups as examples, of as many chunks): one workgroup
// then serves as both, and level 1 takes n_ex workgroups per tile instead of n_ex + G1.
__host__ __device__ inline bool examples_are_groups(const ReduceArgs &a) { return a.n_ex == a.G1 && a.ex_gs == a.gs; }
__host__ __device__ inline int reduce_groups_count(const ReduceArgs &a)
{
    return examples_are_groups(a) ? a.n_ex : a.n_ex + a.G1;
}

// These kernels are a handful of dependent memory round trips long, so every level issues its
// loads in batches of eight before it adds them (in index order: the sums are reproducible).

// ---------------------------------------------------------------------------------------
// The whole reduction in one launch.  A workgroup owns a slab of 4*kQ columns and reads all chunks' sums of it: it
// writes dgamma and dbeta there, and leaves its part of every squared norm; the workgroup that arrives last adds
// those parts up.  Latency bound (three dependent trips to memory); against two levels it saves a launch and the
// trip of the group sums.  Whole backward calls, us, two levels -> this: B=4 T=128 D=256 fp32 12.2 -> 9.5, B=8 T=1024
// D=768 bf16 21.7 -> 18.3, B=8 T=4096 D=8192 284 -> 277, B=8 T=500 D=1001 78.0 -> 48.5 (rows of the workspace that begin at any
// float: read by 16 bytes too, which takes no longer; element by element the call took 16.8 us, so 15.5); the deferred reduction of 48
// layers of B=16 T=2048 D=2048 45.0 -> 38.5.
//
// The parts cross from one XCD's cache to another's without a fence (a release at device scope writes back the
// whole L2, for every workgroup one after the other: the form with fences took longer than the two launches):
// they are stored and loaded by device-scope atomic accesses, which go to the memory that all XCDs share, a
// workgroup waits until its stores are acknowledged there before it counts itself as arrived, and the last one
// loads after it has read the full count.  Every sum has its order from the shape alone, whoever is last.
//
// 512 threads are kWalkers groups of 2*kQ lanes (kQ quads of columns for dgamma, kQ for dbeta).  With fewer examples
// than walkers an example's chunks are split over kWalkers / n_ex of them; otherwise a walker takes a run of whole
// examples, or of chunks when no example's norm is wanted here.
// ---------------------------------------------------------------------------------------
constexpr int kSlabThreads = 512;
__host__ __device__ inline int slab_quads(int D) { return D >= 512 ? 8 : 4; }   // kQ: whole 128-byte lines for wide rows

template <int kLanes>
__device__ __forceinline__ double group_sum_f64(double v)   // over aligned groups of kLanes lanes
{
#pragma unroll
    for (int off = kLanes / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ void store_shared_f64(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_shared_f64(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int kQ>
__device__ __forceinline__ void reduce_slab_body(const ReduceArgs &a, int slab)
{
    constexpr int kCols = 4 * kQ, kLanes = 2 * kQ, kWalkers = kSlabThreads / kLanes, kItems = 2 * kCols;
    constexpr int kUnits = kSlabThreads / kItems;      // walkers or examples combined side by side
    __shared__ double sums[kWalkers][2][kCols];
    __shared__ double totals[kUnits][kItems];
    __shared__ bool last;
    const int tid = threadIdx.x;
    {
        const int walker = tid / kLanes, arr = tid / kQ % 2, quad = tid % kQ;
        const int col = slab * kCols + quad * 4;
        const int left = arr == 0 || a.dbeta ? a.D - col : 0;   // columns this lane has (4 or more: a whole quad)
        const int split = a.n_ex > 0 && a.n_ex <= kWalkers ? kWalkers / a.n_ex : 1;   // walkers per example
        int m0, m1, flush = 0;                                  // chunks of this walker; chunks per example to finish
        if (a.n_ex > 0 && a.n_ex <= kWalkers) {
            const int e = walker / split, part = walker % split, per = (a.ex_gs + split - 1) / split;
            m0 = e < a.n_ex ? e * a.ex_gs + min(part * per, a.ex_gs) : 0;
            m1 = e < a.n_ex ? e * a.ex_gs + min((part + 1) * per, a.ex_gs) : 0;
        } else {
            const int unit = a.n_ex > 0 ? a.ex_gs : 1, n = a.n_slots / unit, per = (n + kWalkers - 1) / kWalkers;
            m0 = min(walker * per, n) * unit;
            m1 = min((walker + 1) * per, n) * unit;
            flush = a.n_ex > 0 ? a.ex_gs : 0;
        }
        double acc[4] = {0, 0, 0, 0}, run[4] = {0, 0, 0, 0};
        const int64_t stride = 2 * (int64_t)a.D;
        const float *base = a.part + (int64_t)arr * a.D + col;
        const bool whole = left >= 4;                           // a quad at any column: rows of the workspace are aligned to a float
        auto finish_example = [&](int e) {
            double q = 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float f = (float)acc[i];                  // an example's gradient as fp32 values, squared in fp64
                q += (double)f * f;
                run[i] += acc[i];
                acc[i] = 0.0;
            }
            q = group_sum_f64<kQ>(q);
            if (quad == 0) store_shared_f64(a.slab + ((int64_t)e * a.nslab + slab) * 2 + arr, q);
        };
        int to_go = flush, e = flush > 0 ? m0 / flush : 0;
        for (int m = m0; m < m1; m += 8) {
            float4 u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float *p = base + min(m + i, m1 - 1) * stride;
                u[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (whole) u[i] = __builtin_bit_cast(float4, (u32x4_t)*(const __attribute__((address_space(1))) u32x4_at4_t *)p);
            }
            if (left > 0 && !whole) {                           // the last quad of a ragged row
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float *p = base + min(m + i, m1 - 1) * stride;
                    u[i].x = p[0];
                    if (left > 1) u[i].y = p[1];
                    if (left > 2) u[i].z = p[2];
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (m + i < m1) {
                    acc[0] += u[i].x; acc[1] += u[i].y; acc[2] += u[i].z; acc[3] += u[i].w;
                    if (flush > 0 && --to_go == 0) {
                        finish_example(e++);
                        to_go = flush;
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) sums[walker][arr][quad * 4 + i] = flush > 0 ? run[i] : acc[i];
    }
    __syncthreads();
    // item = (array, column); the units are the examples when walkers share them, else the walkers
    const int item = tid % kItems, lane0 = tid / kItems, arr = item / kCols, c = item % kCols;
    {
        const bool shared_ex = a.n_ex > 0 && a.n_ex <= kWalkers;
        const int split = shared_ex ? kWalkers / a.n_ex : 1, units = shared_ex ? a.n_ex : kWalkers;
        double total = 0.0;
        for (int e = lane0; e < units; e += kUnits) {
            double v = 0.0;
            for (int j = 0; j < split; ++j) v += sums[e * split + j][arr][c];
            total += v;
            if (shared_ex) {
                const float f = (float)v;
                const double q = group_sum_f64<kCols>((double)f * f);
                if (c == 0) store_shared_f64(a.slab + ((int64_t)e * a.nslab + slab) * 2 + arr, q);
            }
        }
        totals[lane0][item] = total;
    }
    __syncthreads();
    if (tid < kItems) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < kUnits; ++u) v += totals[u][tid];
        const int col = slab * kCols + c;
        float *dst = arr == 0 ? a.dgamma : a.dbeta;
        const bool mine = col < a.D && dst;
        if (mine && a.accumulate) v += (double)dst[col];
        const float f = (float)v;
        if (mine) dst[col] = f;
        const double q = group_sum_f64<kCols>(mine ? (double)f * f : 0.0);     // squares of the values as stored
        if (c == 0) store_shared_f64(a.slab + ((int64_t)a.n_ex * a.nslab + slab) * 2 + arr, q);
    }
    if (a.n_ex == 0 && !a.big_sq) return;
    // every thread: this thread's parts have reached the memory that all XCDs share
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        last = __hip_atomic_fetch_add(a.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)a.nslab - 1u;
    __syncthreads();
    if (!last) return;
    if (tid == 0) __hip_atomic_store(a.arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // sums over the slabs, in an order fixed by the shape: `lanes` threads per sum
    const int nsums = 2 * (a.n_ex + 1);
    int lanes = 16;
    while (lanes > 1 && nsums * lanes > kSlabThreads) lanes >>= 1;
    for (int i = tid / lanes; i < nsums; i += kSlabThreads / lanes) {
        const double *p = a.slab + (int64_t)(i >> 1) * a.nslab * 2 + (i & 1);
        double v = 0.0;
        for (int k = tid % lanes; k < a.nslab; k += lanes * 8) {
            double u[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) u[j] = load_shared_f64(p + 2 * (int64_t)min(k + j * lanes, a.nslab - 1));
#pragma unroll
            for (int j = 0; j < 8; ++j) v += k + j * lanes < a.nslab ? u[j] : 0.0;
        }
        for (int off = lanes / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
        if (tid % lanes == 0) {
            float *dst = i < 2 * a.n_ex ? (i & 1 ? a.pe_beta_sq : a.pe_gamma_sq) : a.big_sq;
            if (dst && (i & 1) && !a.dbeta) dst = nullptr;      // no beta
            if (dst) dst[i < 2 * a.n_ex ? i >> 1 : i & 1] = (float)v;
        }
    }
}

// grid (nslab) for one layer
template <int kQ>
__global__ __launch_bounds__(kSlabThreads) void reduce_slab_kernel(ReduceArgs a)
{
    reduce_slab_body<kQ>(a, blockIdx.x);
}

// Level 1 of two.  grid (ntile, reduce_groups_count), 256 threads: the column tiles of a run of chunks are neighbours in
// launch order, so that the 1 KiB pieces they read of the same chunk vectors are fetched together (with the tiles
// as the slow grid index the batched launch of the 48-layer step took 57 us instead of 35).  A workgroup adds
// the column sums of a run of consecutive chunks: the four waves split the run, add in chunk order, then the
// waves' partial sums are added in wave order.
// The first n_ex workgroups of a tile take one example each and leave the squares of its sums (their sums are
// not kept); the other G1 take one group of chunks each, for the batch gradients.  With a single group the group
// sums ARE the batch gradients and go straight to dgamma / dbeta.
__device__ __forceinline__ void reduce_groups_body(const ReduceArgs &a, int gx, int tile)
{
    __shared__ double wsum[4][8][kWave];   // [wave][array*4 + component][lane]
    __shared__ double slots[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col0 = tile * kTile;

    const bool example = gx < a.n_ex;
    const int g = example ? gx : gx - a.n_ex;
    const int run = example ? a.ex_gs : a.gs;
    const int m0 = g * run, m1 = min(m0 + run, a.n_slots);
    const int per = (m1 - m0 + 3) / 4;
    const int w0 = min(m0 + wave * per, m1), w1 = min(w0 + per, m1);
    const int c4 = col0 + lane * 4;            // this lane's four columns
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (c4 < a.D) {
        const int64_t stride = 2 * (int64_t)a.D;
        if (c4 + 4 <= a.D) {                   // (rows of the workspace are aligned to a float)
            for (int m = w0; m < w1; m += 8) {
                float4 u[8], v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int mm = min(m + i, w1 - 1);
                    const float *p = a.part + mm * stride + c4;
                    using P = const __attribute__((address_space(1))) u32x4_at4_t *;
                    u[i] = __builtin_bit_cast(float4, (u32x4_t)*(P)p);
                    v[i] = __builtin_bit_cast(float4, (u32x4_t)*(P)(p + a.D));
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (m + i < w1) {
                        acc[0] += u[i].x; acc[1] += u[i].y; acc[2] += u[i].z; acc[3] += u[i].w;
                        acc[4] += v[i].x; acc[5] += v[i].y; acc[6] += v[i].z; acc[7] += v[i].w;
                    }
                }
            }
        } else {                               // the last columns of a ragged row: element by element
            const int nc = a.D - c4;
            for (int m = w0; m < w1; ++m) {
                const float *p = a.part + m * stride + c4;
                for (int i = 0; i < nc; ++i) {
                    acc[i] += p[i];
                    acc[4 + i] += p[a.D + i];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) wsum[wave][i][lane] = acc[i];
    __syncthreads();
    // thread -> one column of the tile
    const int col = col0 + tid;
    const int src_lane = tid >> 2, comp = tid & 3;
    double v0 = 0.0, v1 = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        v0 += wsum[w][comp][src_lane];
        v1 += wsum[w][4 + comp][src_lane];
    }
    if (example) {
        // an example's gradient as fp32 values, their squares summed in fp64
        const float f0 = (float)v0, f1 = (float)v1;
        const double e0 = block_sum_f64(col < a.D ? (double)f0 * f0 : 0.0, slots[0]);
        const double e1 = block_sum_f64(col < a.D ? (double)f1 * f1 : 0.0, slots[1]);
        if (tid == 0) {
            a.part_s[((int64_t)g * a.ntile + tile) * 2] = e0;
            a.part_s[((int64_t)g * a.ntile + tile) * 2 + 1] = e1;
        }
        if (!examples_are_groups(a)) return;
    }
    const bool single = a.G1 == 1;
    if (single && a.accumulate && col < a.D) {   // on top of what dgamma / dbeta hold
        v0 += (double)a.dgamma[col];
        if (a.dbeta) v1 += (double)a.dbeta[col];
    }
    const float f0 = (float)v0, f1 = (float)v1;
    if (col < a.D) {
        if (single) {
            a.dgamma[col] = f0;
            if (a.dbeta) a.dbeta[col] = f1;
        } else {
            a.grp[((int64_t)g * 2) * a.D + col] = f0;
            a.grp[((int64_t)g * 2 + 1) * a.D + col] = f1;
        }
    }
    if (single) {
        // squares of the values as stored (fp32), summed in fp64
        const double q0 = block_sum_f64(col < a.D ? (double)f0 * f0 : 0.0, slots[0]);
        const double q1 = block_sum_f64(col < a.D ? (double)f1 * f1 : 0.0, slots[1]);
        if (tid == 0) {
            a.part_big[tile * 2] = q0;
            a.part_big[tile * 2 + 1] = q1;
        }
    }
}

__global__ __launch_bounds__(kTile) void reduce_groups_kernel(ReduceArgs a)
{
    reduce_groups_body(a, blockIdx.y, blockIdx.x);
}

// Sum over the groups for one column (Appendix B steps 3, 7), groups added in order.
__device__ __forceinline__ void sum_groups(const float *grp, int G1, int D, int col, double &s0,
                                           double &s1)
{
    const int64_t stride = 2 * (int64_t)D;
    s0 = s1 = 0.0;
    for (int g = 0; g < G1; g += 8) {
        float u[8], v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float *p = grp + min(g + i, G1 - 1) * stride + col;
            u[i] = p[0];
            v[i] = p[D];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (g + i < G1) {
                s0 += u[i];
                s1 += v[i];
            }
        }
    }
}

// Per-example and batch squared norms from their per-tile parts, tiles added in order.
__device__ __forceinline__ void finish_scalars(const ReduceArgs &a, int tid, int nthreads)
{
    for (int b = tid; b < a.n_ex; b += nthreads) {
        double sg = 0.0, sb = 0.0;
        for (int t = 0; t < a.ntile; ++t) {
            sg += a.part_s[((int64_t)b * a.ntile + t) * 2];
            sb += a.part_s[((int64_t)b * a.ntile + t) * 2 + 1];
        }
        a.pe_gamma_sq[b] = (float)sg;
        if (a.pe_beta_sq) a.pe_beta_sq[b] = (float)sb;
    }
}

// Levels 2 and 3 in ONE workgroup of 1024 threads: dgamma, dbeta, their squared norms, and the
// per-example squared norms.  Used alone when the group sums are small, and one workgroup per
// layer when many layers are finished at once.
__device__ __forceinline__ void reduce_final_body(const ReduceArgs &a)
{
    __shared__ double slots[2][16];
    const int tid = threadIdx.x;
    double q0 = 0.0, q1 = 0.0;
    if (a.G1 > 1) {
        for (int col = tid; col < a.D; col += 1024) {
            double s0, s1;
            sum_groups(a.grp, a.G1, a.D, col, s0, s1);
            if (a.accumulate) {
                s0 += (double)a.dgamma[col];
                if (a.dbeta) s1 += (double)a.dbeta[col];
            }
            const float f0 = (float)s0, f1 = (float)s1;
            a.dgamma[col] = f0;
            if (a.dbeta) a.dbeta[col] = f1;
            q0 += (double)f0 * f0;
            q1 += (double)f1 * f1;
        }
    }
    finish_scalars(a, tid, 1024);
    if (a.big_sq) {
        if (a.G1 > 1) {
            q0 = block_sum_f64(q0, slots[0]);
            q1 = block_sum_f64(q1, slots[1]);
        } else if (tid < 2) {   // level 1 already left the per-tile parts
            double t2 = 0.0;
            for (int t = 0; t < a.ntile; ++t) t2 += a.part_big[t * 2 + tid];
            if (tid == 0) q0 = t2;
            else q1 = t2;
        }
        if (tid == 0) a.big_sq[0] = (float)q0;
        if (tid == (a.G1 > 1 ? 0 : 1) && a.dbeta) a.big_sq[1] = (float)q1;   // one norm without beta
    }
}

__global__ __launch_bounds__(1024) void reduce_final_small_kernel(ReduceArgs a)
{
    reduce_final_body(a);
}

// Many layers at once (deferred reduction).  Every layer's workspace starts with a DeferHeader
// and has the same layout, because the layers have the same shape.
constexpr int kBatchMax = 64;
struct BatchArgs {
    char *ws[kBatchMax];
    int n;
    int D;
    int ntile;
    int nslab;
    size_t off_grp, off_part_s, off_part_big, off_part;
};

__device__ __forceinline__ ReduceArgs batch_layer_args(const BatchArgs &b, int layer, bool &one_pass)
{
    char *ws = b.ws[layer];
    DeferHeader *head = reinterpret_cast<DeferHeader *>(ws);
    const DeferHeader h = *head;
    one_pass = h.one_pass != 0;
    ReduceArgs a;
    a.nslab = b.nslab;
    a.slab = reinterpret_cast<double *>(ws + b.off_grp);
    a.arrived = &head->arrived;
    a.part = reinterpret_cast<const float *>(ws + b.off_part);
    a.grp = reinterpret_cast<float *>(ws + b.off_grp);
    a.part_s = reinterpret_cast<double *>(ws + b.off_part_s);
    a.part_big = reinterpret_cast<double *>(ws + b.off_part_big);
    a.dgamma = h.dgamma; a.dbeta = h.dbeta;
    a.pe_gamma_sq = h.pe_gamma_sq; a.pe_beta_sq = h.pe_beta_sq; a.big_sq = h.big_sq;
    a.n_slots = h.n_slots; a.gs = h.gs; a.G1 = h.G1; a.n_ex = h.n_ex; a.ex_gs = h.ex_gs; a.D = b.D; a.ntile = b.ntile;
    a.accumulate = h.accumulate;
    return a;
}

// grid (nslab, layers)
template <int kQ>
__global__ __launch_bounds__(kSlabThreads) void reduce_slab_batch_kernel(BatchArgs b)
{
    bool one_pass;
    const ReduceArgs a = batch_layer_args(b, blockIdx.y, one_pass);
    if (one_pass) reduce_slab_body<kQ>(a, blockIdx.x);
}

// grid (ntile, most examples + groups of any layer, layers): workgroups beyond a layer's own count leave at once
__global__ __launch_bounds__(kTile) void reduce_groups_batch_kernel(BatchArgs b)
{
    bool one_pass;
    const ReduceArgs a = batch_layer_args(b, blockIdx.z, one_pass);
    if (one_pass || (int)blockIdx.y >= reduce_groups_count(a)) return;
    reduce_groups_body(a, blockIdx.y, blockIdx.x);
}

// grid (layers)
__global__ __launch_bounds__(1024) void reduce_final_batch_kernel(BatchArgs b)
{
    bool one_pass;
    const ReduceArgs a = batch_layer_args(b, blockIdx.x, one_pass);
    if (one_pass) return;
    if (a.G1 == 1 && a.n_ex == 0 && !a.big_sq) return;
    reduce_final_body(a);
}

// The same two levels for shapes whose layers are nearly always reduced in one launch, but may have been cut for two
// levels (other pointers, a plain call).  A workgroup takes every gridDim.y-th of a layer's examples and groups, at most
// kBatchGroups workgroups to a column tile: one for each of hundreds of examples took some 10 us to come and go in
// vain.  The slabs of the others share the launch of the second level.  16 layers, us, two levels / slabs and two levels
// one after the other / this: bf16 B=512 T=64 D=1024 24 / 33 / 19, D=2048 40 / 55 / 30, B=1000 T=33 D=768 31 / 45 / 25.
constexpr int kBatchGroups = 64;
__global__ __launch_bounds__(kTile) void reduce_groups_few_batch_kernel(BatchArgs b)
{
    bool one_pass;
    const ReduceArgs a = batch_layer_args(b, blockIdx.z, one_pass);
    if (one_pass) return;
    const int n = reduce_groups_count(a);
    for (int g = blockIdx.y; g < n; g += gridDim.y) {
        if (g != (int)blockIdx.y) __syncthreads();             // the last one's sums in LDS have been read
        reduce_groups_body(a, g, blockIdx.x);
    }
}

// grid (nslab, layers): a slab of a layer that is reduced in one launch (by half of the waves, the others end at once), or,
// by its first workgroup, the second level of one that is not.
template <int kQ>
__global__ __launch_bounds__(1024) void reduce_last_batch_kernel(BatchArgs b)
{
    bool one_pass;
    const ReduceArgs a = batch_layer_args(b, blockIdx.y, one_pass);
    if (one_pass) {
        if (threadIdx.x < kSlabThreads) reduce_slab_body<kQ>(a, blockIdx.x);
        return;
    }
    if (blockIdx.x > 0 || (a.G1 == 1 && a.n_ex == 0 && !a.big_sq)) return;
    reduce_final_body(a);
}

// Level 2 for large shapes: grid ntile, 256 threads, one column per thread.
__global__ __launch_bounds__(kTile) void reduce_final_tiles_kernel(ReduceArgs a)
{
    __shared__ double slots[2][4];
    const int tid = threadIdx.x, tile = blockIdx.x;
    const int col = tile * kTile + tid;
    double s0 = 0.0, s1 = 0.0;
    if (col < a.D) {
        sum_groups(a.grp, a.G1, a.D, col, s0, s1);
        if (a.accumulate) {
            s0 += (double)a.dgamma[col];
            if (a.dbeta) s1 += (double)a.dbeta[col];
        }
        a.dgamma[col] = (float)s0;
        if (a.dbeta) a.dbeta[col] = (float)s1;
    }
    const double d0 = (double)(float)s0, d1 = (double)(float)s1;
    const double q0 = block_sum_f64(d0 * d0, slots[0]);
    const double q1 = block_sum_f64(d1 * d1, slots[1]);
    if (tid == 0) {
        a.part_big[tile * 2] = q0;
        a.part_big[tile * 2 + 1] = q1;
    }
}

// Level 3 for large shapes: one workgroup.
__global__ __launch_bounds__(256) void reduce_scalars_kernel(ReduceArgs a)
{
    const int tid = threadIdx.x;
    finish_scalars(a, tid, 256);
    if (a.big_sq && tid < (a.dbeta ? 2 : 1)) {
        double t2 = 0.0;
        for (int t = 0; t < a.ntile; ++t) t2 += a.part_big[t * 2 + tid];
        a.big_sq[tid] = (float)t2;
    }
}

// Section 2.1 Eq. 3-5 with B_small = 1, B_big = B; one workgroup.
__global__ __launch_bounds__(256) void gns_estimate_kernel(const float *pe_sq, const float *big_sq,
                                                           int n_groups, int B, float pe_scale,
                                                           float *out)
{
    __shared__ double slots[2][4];
    const int64_t n = (int64_t)n_groups * B;
    double s = 0.0, g = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) s += (double)pe_sq[i];
    for (int i = threadIdx.x; i < n_groups; i += blockDim.x) g += (double)big_sq[i];
    s = block_sum_f64(s, slots[0]);
    g = block_sum_f64(g, slots[1]);
    if (threadIdx.x == 0) {
        const double Bd = (double)B, c = (double)pe_scale;
        const double small = c * c * (s / Bd);  // mean over examples, then the correction
        const double big = g;
        const double G2 = (Bd * big - small) / (Bd - 1.0);   // Eq. 4 with B_small = 1
        const double S = (small - big) / (1.0 - 1.0 / Bd);   // Eq. 5 with B_small = 1
        out[0] = (float)small;
        out[1] = (float)big;
        out[2] = (float)G2;
        out[3] = (float)S;
        out[4] = (float)(S / G2);                            // Eq. 3
    }
}

}  // namespace lnpegn
