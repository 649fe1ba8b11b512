// C ABI of the lnpegn library (declared in include/lnpegn.h): argument validation, launch
// planning and kernel launches.  No allocation, no synchronisation, no state between calls
// apart from the process-wide launch-shape overrides of lnpegn_set_tuning() and the per-device
// address of the fixed scratch of ln_bwd_pegn_static.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/lnpegn.h"
#include "lnpegn_finalize.h"
#include "lnpegn_tracker.h"
#include "lnpegn_launch.h"
#include "lnpegn_rows.h"

// Scratch of ln_bwd_pegn_static: the workspace of a backward call, held by the library itself so that the
// call allocates nothing.  One copy per GPU the library runs on, kept until the process ends.  In host
// code this name is only a handle for hipGetSymbolAddress; kernels are given the address it returns.
constexpr size_t kStaticScratchBytes = LNPEGN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace lnpegn {
thread_local int g_last_hip_error = 0;   // hipError_t behind this thread's latest LNPEGN_EHIP from a row kernel launch
extern int g_emb_run_blocks;   // embedding_pegn.hip: workgroups of its run kernel per column group
namespace {

// launch-shape overrides (0 = automatic)
int g_chunks_pegn = 0;
int g_chunks_plain = 0;
int g_waves = 0;
int g_vpt_max = 0;          // cap on 16-byte vectors per lane and array (0: automatic)
int g_xcd = -1;        // hand neighbouring chunks to the same XCD: 0 never, 1 always, -1 automatic
int g_blocked = -1;    // chunks of consecutive rows: 0 never, 1 always, -1 automatic
int g_dx_cached = -1;  // dx stores write-back instead of streaming: 0 never, 1 always, -1 automatic
bool g_overridden = false;   // an override has been set in this process: layers may have been launched under any plan
int g_stagger = -1;   // rows between the sweep starts of consecutive examples (-1 = automatic)
// one-shot profiling events around the row kernel (null = disarmed)
hipEvent_t g_ev_start = nullptr;
hipEvent_t g_ev_stop = nullptr;

constexpr int kMaxChunks = 16384;
constexpr int kCUs = 256;           // MI355X
constexpr int kGroups = 16;         // groups of chunks in the reduction that gives the batch gradients
constexpr int64_t kSmallFinal = 32768;  // G1*D up to which one workgroup finishes the reduction
constexpr int kSlabChunks = 2048;   // most chunks for the reduction in one launch
constexpr int kSlabParts = 8192;    // ... most parts (examples times slabs) of the per-example norms
constexpr int kSlabExamples = 64;   // ... and most examples
constexpr size_t kAlign = 256;

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct Plan {
    // row kernel
    bool plain;       // no per-example outputs: the plain backward's kernel
    bool fast;        // vectorised kernels
    bool ragged;      // ... in their form for rows of any width and address
    bool sync;        // several waves per row
    int vpt;          // 16-byte vectors per lane
    int S, R;         // waves per row, row groups per workgroup
    int max_threads;  // launch bound of the instantiation
    int nvec;
    int64_t Tp;       // rows per partition example
    int C;            // chunks per partition example
    int64_t n_slots;  // chunks in all
    int rows_per;     // > 0: a chunk is a block of that many consecutive rows; 0: every C-th row of its example
    int64_t stagger;  // rows between the sweep starts of consecutive examples
    int xcd_chunks;   // > 0: chunks per XCD (an example's chunks share an L2); 0: chunks in launch order
    size_t lds_bytes;
    // reduction
    int ntile;
    int gs, G1;       // chunks per group, groups
    bool emit_pe;     // row kernel writes the per-example norms (a chunk is a whole example)
    int n_ex;         // examples whose norms the reduction takes from their chunks' sums (0 or B)
    bool one_pass;    // reduced by the slab kernel, else in two levels
    int nslab;
    // workspace layout (byte offsets); everything but `part` depends on B and D only, so that a
    // batched reduction can address any layer of the same shape
    size_t off_grp, off_part_s, off_part_big, off_part, total;
};
constexpr size_t kHeaderBytes = 256;

// Chunks per example, given W workgroups resident at a time.  W/B of them fill one round of workgroups when B
// divides W; when they would leave much of a round empty (B*C/W below 0.85, or a last round that is less than a
// third full), the example is cut finer, into three rounds or more: many short workgroups even out by themselves,
// at the price of one more flush of column sums per chunk.  Measured, bf16 D=1024, us per launch, W/B chunks ->
// this choice: B=300 T=100 39.6 -> 33.3, B=260 T=128 44.6 -> 38.6, B=600 T=64 47.7 -> 45.5, B=513 T=64
// 40.0 -> 37.0, B=384 T=64 30.0 -> 29.1, B=200 T=128 31.4 -> 30.2; D=2048: B=300 T=100 104.5 -> 77.9, B=600 T=64
// 105.3 -> 91.5; D=4096: B=300 T=100 170.1 -> 153.5.  (B=700 T=48 and B=1000 T=32, whose second round is more
// than a third full, are faster with one chunk per example: 35.8 against 36.9 and 34.1 against 35.2.)
int64_t chunks_per_example(int64_t B, int64_t T, int64_t W, int R)
{
    const int64_t c0 = W / B > 1 ? W / B : 1;
    const int64_t n = B * c0, full = n / W, rest = n % W;   // rounds that are full, workgroups in the last one
    const bool fits = n <= W ? 20 * n >= 17 * W
                             : rest == 0 || full >= 3 || (full == 1 && 10 * rest >= 3 * W);
    if (fits) return c0;
    const int64_t c3 = (3 * W + B - 1) / B;         // three rounds
    return (c3 <= 16 && T / c3 >= (R > 4 ? 4 * R : 16)) ? c3 : c0;    // ... unless that leaves a chunk fewer than 16 rows, or four for
                                                                      // each of more than four row groups
}

// What the pointers of a call allow: nothing but element accesses, vectors at element addresses, aligned vectors.
enum Access { kGenericAccess, kElementAccess, kVectorAccess };

Plan make_plan(int B, int T, int D, lnpegn_dtype dt, bool pegn, Access access)
{
    Plan p{};
    p.plain = !pegn;
    const int E = dt == LNPEGN_BF16 ? 8 : 4;
    const int64_t N = (int64_t)B * T;
    int vpt_max = 16 / E;                            // 16 elements per lane ...
    if (g_vpt_max > 0 && g_vpt_max < vpt_max) vpt_max = g_vpt_max;
    // ... up to 32 for rows beyond eight waves of 16 (D > 8192): eight waves of 24 or 32 elements per lane
    if (D % E == 0 && D / E > 64 * vpt_max * 8) vpt_max = 32 / E;
    p.fast = access == kVectorAccess && (D % E == 0) && (D / E <= 64 * vpt_max * 8);
    // Other widths and addresses: the same kernels with unaligned vectors, for rows of one vector up to eight waves of
    // 16 elements per lane; narrower and wider ones take the generic kernel.
    p.ragged = !p.fast && access != kGenericAccess && D >= E && ceil_div(D, E) <= 64 * vpt_max * 8 && vpt_max <= 16 / E;
    p.fast = p.fast || p.ragged;
    p.nvec = p.fast ? ceil_div(D, E) : 0;
    p.sync = false;
    p.vpt = 1;
    p.S = 1;
    p.R = 4;
    p.max_threads = 256;
    int waves_per_simd = 4;                          // resident waves per SIMD to aim for
    const bool uneven = pegn && B < kCUs && 20 * (kCUs / B * B) < 17 * kCUs;    // one workgroup a CU does not come out even
    if (p.fast) {
        p.S = vpt_max > 16 / E ? 8 : ceil_div(p.nvec, 64 * vpt_max);   // beyond 16 elements per lane: always eight waves
        p.vpt = ceil_div(p.nvec, 64 * p.S);
        p.sync = p.S > 1;
        const int elems = p.vpt * E;                 // per lane
        waves_per_simd = elems > 8 ? 2 : 4;          // measured: more waves of 16-element lanes only add contention
        // Narrow lanes, rows of one wave: half as many workgroups (512) where what the reduction saves is more than the
        // row kernel loses: in short tensors, and in longer ones if the fewer waves still keep as many bytes under way as the memory
        // wants, with lanes of one vector that are (nearly) all full or lanes of two.  Times with 1024 as multiples of those with 512,
        // N = B*T of 8000 / 12000 / 24000 / 64000, forward and backward, B=16: bf16 D=64 1.06 / 1.03 / 0.94 / 0.90, D=256 1.08 / 1.07 /
        // 0.91 / 0.83, fp32 D=200 1.05 / 1.01 / 0.90 / 0.90, D=416 1.09 / 1.08 / 0.99 / 1.06, D=512 1.10 / 1.10 / 1.02 / 1.03.  Of one vector
        // a lane the fewer the rows the less full the lanes, and fp32, whose lanes do half the work for their bytes, less than bf16.  Medians of
        // 2250 calls of random B up to 32 and T, backward with norms, N to 20000 / 24576 / 32768 / 40000 / 64000 / beyond: bf16 57 to 63
        // vectors 1.05 / 1.05 / 1.03 / 1.01 / 0.98 / 0.98, fp32 0.99 / 0.99 / 0.98 / 0.98 / 0.97 / 0.95, 49 to 56 0.97 / 0.94 (to 16384 1.02);
        // 64 vectors, means, 1.06 / 1.06 / 1.03 / 1.03 / 1.02 / 1.01 (bf16 63 beyond 40000 1.06), and bf16 49 to 56 1.05 to 20000, 1.01 to 28000, 0.99 to 40000.
        const int64_t longest = p.nvec >= (E == 8 ? 63 : 64) ? N : E == 4 ? 16384 : p.nvec >= 57 ? 40960 : 24576;
        if (p.S == 1 && elems <= 8 && (!pegn || B <= 32) && N >= 8192 && (N <= 12288 || (p.nvec > 48 * p.vpt && N <= longest)))
            waves_per_simd = 2;
        // launch bound of the instantiation that will run: 256 threads for S = 1, 2, 4; 512 else
        const int max_waves = (elems <= 8 && (p.ragged ? p.S == 1 : p.S <= 2)) ? 4 : 8;
        // row groups per workgroup.  Wide lanes: six waves per workgroup, one workgroup per CU (measured, B*T =
        // 32768 rows: bf16 D=2048 69.2 -> 66.9 us per-example and 69.0 -> 65.4 plain against four waves; fp32
        // D=2048 151.7 -> 145.6 and 133 -> 131; eight waves are slower than six; no difference where a row
        // already takes four or eight waves).
        // Rows that one wave covers, wide lanes: eight row groups, one workgroup per CU, as soon as a chunk has two rows
        // for each.  The same waves as with two workgroups of four, but half the chunks, whose column sums the reduction
        // reads back.  us a call, row kernel + reduction, four / eight: bf16 B=8 T=1024 D=768 9.8 + 8.2 / 9.2 + 6.3, B=16 T=2048
        // D=768 27.7 + 8.1 / 27.0 + 7.0, B=8 T=500 D=1001 9.6 + 11.5 / 8.3 + 8.5, B=48 T=256 D=768 14.6 + 8.1 / 14.0 + 6.9, B=100
        // T=24 15.5 / 12.3, fp32 B=16 T=2048 D=1024 68.7 + 15.6 / 68.7 + 11.5; T=24 B=8 11.0 / 11.4; plain B=8 T=1024 D=768
        // 9.8 + 6.2 / 9.1 + 4.6.  Many examples in long tensors, whose chunks come from rounds of workgroups, stay at four.
        // Nor do those whose examples don't divide the CUs, unless each is one chunk: two workgroups a CU then, which fp32 and ragged
        // rows take no better than four smaller ones and bf16 rows only if the examples are long enough for as many.  As multiples of the
        // time with four, deferred calls: fp32 D=1024 B=100 T=60 1.12, B=150 T=50 1.04, B=120 T=60 (even) 0.93, B=100 T=24 0.86; D=768 B=90
        // T=60 1.10; bf16 D=1001 B=90 T=60 1.15, D=768 1.03, B=100 T=100 0.97.  And fp32 or ragged rows of 48 to 79 examples that
        // are one chunk are too few: fp32 D=1024 B=64 T=27 1.21, D=768 1.08, bf16 D=1001 1.11.
        const bool sturdy = E == 8 && !p.ragged;
        const bool two = uneven && T >= 32 && !(sturdy && T / 16 >= 2 * kCUs / B);
        const bool thin = pegn && !sturdy && T < 32 && B >= 48 && B < 80;
        const bool eight = (!pegn || B <= 32 || N <= 16384) && (pegn ? T : N) >= 16 && !two && !thin;
        // (fp32 rows of four waves: two row groups, measured with the per-example sweeps, 288.7 -> 273.8 us)
        // (rows of two waves with lanes left over, D=1280, 1536 or 1600 in bf16, have fewer bytes in flight per
        // wave and take four row groups: D=1280 64.5 -> 52.0 us, D=1536 65.0 -> 55.3; rows of three waves take two:
        // bf16 D=3072 147.7 -> 111.5 per-example and 107.6 -> 100.3 plain, fp32 D=3072 216.3 -> 205.1)
        const bool full = !p.ragged && p.nvec == 64 * p.S * p.vpt;
        int R = g_waves > 0 ? g_waves / p.S
                : (elems > 8 && p.S == 2) ? (full ? 3 : 4)
                : p.S == 3 ? 2
                : (pegn && E == 4 && p.S == 4 && p.vpt >= 3) ? 2
                : (elems > 8 && p.S == 1 && eight) ? 8
                : (p.S >= 4 ? 1 : 4 / p.S);
        if (R < 1) R = 1;
        while (R > 1 && R * p.S > max_waves) --R;
        p.R = R;
        p.max_threads = 64 * max_waves;
    }
    const int nwaves = p.fast ? p.R * p.S : 4;
    // one full round of resident workgroups unless told otherwise
    int target = pegn ? g_chunks_pegn : g_chunks_plain;
    if (target <= 0) {
        int per_cu = (waves_per_simd * 4) / nwaves > 0 ? (waves_per_simd * 4) / nwaves : 1;
        // Per-example sweeps, measured on B*T = 32768 rows (bf16, us per launch, fewer / more chunks):
        //   rows of one wave   (D=768: 34.8 / 29.3, D=1024: 39.6 / 38.8)    two workgroups of four waves per CU
        //   rows of two waves  (D=2048: six waves per workgroup)             one workgroup per CU
        //   rows of four waves (D=4096: 138.9 / 147.8)                       one workgroup per CU: half as many
        //       chunks per example keep each example's moving window of memory half as wide
        //   rows of eight waves (D=8192: 279.6 / 268.0)                      two rounds of workgroups: the second
        //       round starts where the first finishes, which evens out the CUs' unequal memory throughput
        // ... as long as a chunk keeps a hundred rows or so (short launches want the parallelism more).
        if (pegn && p.fast && p.S == 4 && waves_per_simd == 2 && per_cu > 1 && !(E == 4 && p.vpt >= 3) &&
            N / ((int64_t)kCUs * (per_cu / 2)) >= 96)
            per_cu /= 2;
        //   fp32 rows of two and four waves (lanes of four vectors; D=2048: 140.5 / 137.9, D=4096 with two row
        //       groups: 290.8 / 273.8) also take two rounds
        const bool wide_f32 = E == 4 && p.vpt >= 3 && p.S >= 2;
        //   rows of six and seven waves likewise (bf16 D=6144: 224.6 / 216.9)
        if (pegn && p.fast && (p.S >= 6 || wide_f32) && N / ((int64_t)kCUs * 2) >= 32) per_cu = 2;
        target = kCUs * per_cu;
    }
    // rows per chunk at least: two per row group, and four in all -- a chunk ends with a write of its 2*D column
    // sums, which is as many bytes as four bf16 rows carry
    const int rows_min = p.fast ? (2 * p.R > 4 ? 2 * p.R : 4) : 4;
    const int R = p.fast ? p.R : 1;
    // Prefer a chunk count that gives every chunk the same number of rows, a multiple of R: no
    // partial last iteration.  Searched downwards, never below 3/4 of the first choice.  Eight row groups, one workgroup a CU:
    // not where the fewer workgroups iterate more often than the first choice.  Deferred calls, as multiples of the time with four
    // row groups, searched so / this: bf16 D=768 B=5 T=9672 (39 chunks for 51) 1.06 / 0.99, D=568 B=4 T=16000 (50 for 64) 1.16 / 0.98.
    auto even_chunks = [&](int64_t c, int64_t rows) {
        for (int64_t t = c; t >= 1 && 4 * t >= 3 * c; --t)
            if (rows % (t * R) == 0) return R == 8 && rows / (t * R) > (rows - 1) / (c * R) + 1 ? c : t;
        return c;
    };
    if (pegn) {
        p.Tp = T;
        // Eight row groups: where one workgroup per CU does not come out even, two (they fit side by side).  us a call, one / two:
        // bf16 D=768 B=130 T=126 28.0 / 25.8, B=100 T=160 25.8 / 25.4, B=90 T=180 27.1 / 25.2 (B=50 T=300, even, 22.0 / 23.2).
        int64_t c = g_chunks_pegn > 0 || !p.fast ? target / B : chunks_per_example(B, T, p.R == 8 && uneven ? 2 * target : target, p.R);
        // Long launches over fp32 rows of 16 elements per lane: several rounds of shorter workgroups, which even
        // out the CUs' unequal progress (measured, us per launch, one round -> this: B=16 T=2048 D=2048
        // 138.3 -> 134.3, B=8 T=4096 D=2048 137.2 -> 134.2, B=16 T=4096 D=2048 280.9 -> 265.9, B=16 T=2048 D=1024
        // 75.2 -> 72.0, B=16 T=2048 D=4096 279.6 -> 265.1 with two rounds and 283.3 with four; half as many rows,
        // B=16 T=1024 D=2048, are faster in one round, 72.8 against 74.0, and so are bf16 rows: D=2048 68.8 -> 71.2
        // with two rounds).
        // (fp32 D=1280 96.4 -> 93.1, D=1536 112.3 -> 109.2)
        if (g_chunks_pegn <= 0 && p.fast && E == 4 && p.vpt >= 3 && p.S <= 4 && N >= 32768 && B * c <= target) {
            int64_t rounds = p.S == 4 ? 2 : 4;
            while (rounds > 1 && T / (c * rounds) < 16) rounds /= 2;
            c *= rounds;
        }
        const int64_t cmax = T / rows_min > 1 ? T / rows_min : 1;
        if (c > cmax) c = cmax;
        if (c < 1) c = 1;
        p.C = (int)even_chunks(c, T);
        p.n_slots = (int64_t)B * p.C;
        // A chunk that is a whole short example, two or more of them per CU, rows of one wave: eight rows at a
        // time (measured, bf16 D=1024: B=512 T=64 35.8 -> 35.0 us, B=1024 T=32 35.2 -> 34.1, B=700 T=48
        // 37.8 -> 35.7; fp32 B=512 T=64 D=1024 77.5 -> 73.9; with fewer examples than that four rows are faster).
        if (p.fast && g_waves <= 0 && p.C == 1 && p.S == 1 && p.vpt * E > 8 && B >= 2 * kCUs && T >= 32) p.R = 8;
    } else {
        p.Tp = N;
        int64_t c = target;
        const int64_t cmax = N / rows_min > 1 ? N / rows_min : 1;
        if (c > cmax) c = cmax;
        p.C = (int)even_chunks(c, N);
        p.n_slots = p.C;
    }
    // The chunks of an example take every C-th row each, so that together they sweep the example as one narrow
    // window of memory: the fastest pattern as long as the examples, i.e. the windows, are few.  With more than 32
    // examples every chunk takes a block of consecutive rows instead: a few percent behind the best case of
    // the other pattern but without its bad cases (measured, us per launch, every C-th row / blocks: bf16 D=2048,
    // B*T = 32768: B=16 67.5 / 73.6, B=32 70.6 / 73.8, B=64 89.7 / 73.8; D=1024: B=64 48.9 / 37.3, B=128
    // 41.3 / 36.0, B=256 35.2 / 36.0).  The plain backward always has one window (D=2048: 67.3 / 73.2).
    const bool blocked = g_blocked >= 0 ? g_blocked != 0 : pegn && B > 32;
    p.rows_per = (blocked && p.C > 1) ? ceil_div(p.Tp, p.C) : 0;
    // Every example's sweep starts 5T/4B rows after its predecessor's; none when that is less than a row (measured
    // with a chunk per example, bf16 D=1024, no shift / one row: B=512 T=128 76.0 / 96.3 us, B=260 T=128 44.7 / 50.9,
    // B=1000 T=32 35.2 / 39.4, B=512 T=64 36.1 / 35.8).
    p.stagger = g_stagger >= 0 ? (pegn ? g_stagger : 0) : (!pegn || p.rows_per > 0) ? 0 : 5 * (int64_t)T / (4 * (int64_t)B);
    // measured: grouping an example's chunks on one XCD helps wide rows (S >= 4) and is neutral otherwise
    const bool xcd = g_xcd >= 0 ? g_xcd != 0 : p.S >= 4;
    p.xcd_chunks = (xcd && p.fast && p.n_slots % 8 == 0 && p.n_slots / 8 <= INT32_MAX) ? (int)(p.n_slots / 8) : 0;
    {
        const int nw = p.fast ? p.R * p.S : 4;
        const size_t xchg = (size_t)((10 * nw + 2 * p.S + 3) & ~3) * sizeof(float);
        const size_t merge = p.fast && p.R > 1 ? (size_t)nw * 2 * p.vpt * E * kWave * sizeof(float) : 0;
        p.lds_bytes = xchg + (merge > 512 ? merge : 512);
    }
    p.emit_pe = pegn && p.fast && !p.ragged && p.C == 1;
    p.n_ex = pegn && !p.emit_pe ? B : 0;
    p.gs = ceil_div(p.n_slots, kGroups);
    p.G1 = ceil_div(p.n_slots, p.gs);
    p.ntile = ceil_div(D, kTile);
    p.nslab = ceil_div(D, 4 * slab_quads(D));
    // The slab kernel's workgroups are as many as slabs, each reads its columns of every chunk, and the last one adds
    // up nslab parts of every norm.  Few chunks and few norms: one launch.  Many: two levels.  Measured, us a call, two
    // levels / one launch: 64 examples (B=64 T=512 D=1024 bf16) 48.1 / 46.9, 128 (B=128 T=256) 48.3 / 49.7, 200 in 1600
    // chunks (B=200 T=128) 44.8 / 51.1; 8192 parts (B=32 T=300 D=8192) 108.2 / 103.3; 2048 chunks (B=16 T=2048 D=2048
    // fp32) 157.5 / 153.6.  More than 32 examples, of which a walker then takes several: bf16 B=40 D=512 in 1000
    // chunks (T=512) 23.5 / 26.8, D=640 27.4 / 27.0, D=768 28.9 / 28.4; D=256 in 320 chunks (T=64) 13.1 / 11.4; B=33 to 64,
    // D=64 to 512: two levels 0 to 2.2 more up to 512 chunks, 0 to 4.5 less from 825 on; fp32 B=64 T=512 D=768 in 2048 63.0 /
    // 66.1.  Whole-example chunks (T=16)
    // of too few slabs for their number: bf16 D=768 B=1024 27.5 / 26.7, 1536 37.0 / 37.7, 2048 43.4 / 45.1, D=1536
    // B=2048 79.0 / 79.4, D=2048 100.1 / 96.9, fp32 D=256 B=2048 29.8 / 31.8, D=128 23.9 / 23.2.  The parts lie
    // where the two levels keep their group sums.
    const bool many_ex_ok = p.n_ex <= 32 || (p.n_slots <= 1024 && (D >= 640 || p.n_slots <= 640));
    const bool many_chunks_ok = !p.emit_pe || p.n_slots <= 1024 || D <= 192 || D >= 1536;
    p.one_pass = p.n_slots <= kSlabChunks && p.n_ex <= kSlabExamples && many_ex_ok && many_chunks_ok && (int64_t)p.n_ex * p.nslab <= kSlabParts &&
                 (size_t)(p.n_ex + 1) * p.nslab * 2 * sizeof(double) <= (size_t)kGroups * 2 * D * sizeof(float);
    const size_t vec_bytes = (size_t)2 * D * sizeof(float);
    size_t off = kHeaderBytes;            // the layout up to `part` does not depend on the path taken
    p.off_grp = off;       off += align_up((size_t)kGroups * vec_bytes);
    p.off_part_s = off;    off += align_up((size_t)B * p.ntile * 2 * sizeof(double));
    p.off_part_big = off;  off += align_up((size_t)p.ntile * 2 * sizeof(double));
    p.off_part = off;      off += align_up((size_t)p.n_slots * vec_bytes);
    p.total = off;
    return p;
}

bool shape_ok(int B, int T, int D) { return B > 0 && T > 0 && D > 0; }

// Device address of `scratch` on the current device, looked up once per device and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

hipError_t static_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % kAlign) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
bool dtype_ok(int dt) { return dt == LNPEGN_F32 || dt == LNPEGN_BF16; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
Access access_of(const void *x, const void *dy, const void *dx, const void *gamma, int dt)
{
    if (aligned16(x) && aligned16(dy) && aligned16(dx) && aligned16(gamma)) return kVectorAccess;
    const uintptr_t any = reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy) |
                          reinterpret_cast<uintptr_t>(dx) | reinterpret_cast<uintptr_t>(gamma);
    return (any & (dt == LNPEGN_BF16 ? 1u : 3u)) == 0 ? kElementAccess : kGenericAccess;
}

int run_bwd(bool pegn, bool defer, bool accumulate, bool rms, const void *x, const void *dy, const void *gamma, const float *mean,
            const float *rstd, void *dx, float *dgamma, float *dbeta, float *pe_gamma_sq,
            float *pe_beta_sq, float *big_sq, int B, int T, int D, int dt, int gamma_dt, float eps,
            void *workspace, size_t workspace_bytes, void *stream)
{
    if (!shape_ok(B, T, D) || !(eps >= 0.f)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt) || !dtype_ok(gamma_dt)) return LNPEGN_EUNSUPPORTED;
    if (!x || !dy || !gamma || !dx || !dgamma || (!rms && !dbeta)) return LNPEGN_EINVAL;
    if (pegn && (!pe_gamma_sq || (!rms && !pe_beta_sq))) return LNPEGN_EINVAL;
    if (!rms && (mean == nullptr) != (rstd == nullptr)) return LNPEGN_EINVAL;
    if (dx == x) return LNPEGN_EINVAL;
    if ((int64_t)B * T > INT32_MAX) return LNPEGN_EINVAL;   // row indices are 32-bit
    Plan p = make_plan(B, T, D, (lnpegn_dtype)dt, pegn, access_of(x, dy, dx, gamma, dt));
    // (ragged rows may be cut into more chunks than the generic kernel asks for: in less workspace they take that one)
    if (p.ragged && workspace_bytes < p.total) p = make_plan(B, T, D, (lnpegn_dtype)dt, pegn, kGenericAccess);
    if (!workspace || workspace_bytes < p.total) return LNPEGN_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return LNPEGN_EINVAL;
    if (p.n_slots > INT32_MAX) return LNPEGN_EINVAL;

    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    float *part = reinterpret_cast<float *>(ws + p.off_part);

    RowArgs a{};
    a.x = x; a.dy = dy; a.gamma = gamma; a.mean = mean; a.rstd = rstd; a.dx = dx;
    a.part = part; a.pe_gamma_sq = pe_gamma_sq; a.pe_beta_sq = pe_beta_sq;
    a.Tp = p.Tp; a.C = p.C; a.D = D; a.nvec = p.nvec;
    a.rows_per = p.rows_per; a.stagger = p.stagger; a.xcd_chunks = p.xcd_chunks;
    a.S = p.S; a.gamma_is_f32 = gamma_dt == LNPEGN_F32; a.emit_pe = p.emit_pe; a.rms = rms;
    a.eps = eps; a.inv_D = 1.0f / (float)D;
    a.head = reinterpret_cast<DeferHeader *>(ws);
    a.hdr = DeferHeader{dgamma, dbeta, pe_gamma_sq, pe_beta_sq, pegn ? big_sq : nullptr,
                        (int)p.n_slots, p.gs, p.G1, p.n_ex, p.C, accumulate ? 1 : 0, p.one_pass ? 1 : 0, 0u};

    const bool saved = rstd != nullptr;
    const RowLaunch rl{s, g_ev_start, g_ev_stop};
    g_ev_start = g_ev_stop = nullptr;
    RowShape rs{};
    rs.plain = p.plain; rs.fast = p.fast; rs.ragged = p.ragged; rs.vpt = p.vpt; rs.S = p.S; rs.R = p.R; rs.nvec = p.nvec;
    rs.n_slots = p.n_slots; rs.lds_bytes = p.lds_bytes;
    // measured (size of dx in MiB: streaming / write-through, us per launch, one layer at a time): 32: 23.2 / 22.1,
    // 64: 39.1 / 36.6 and 41.2 / 35.9, 96: 57.3 / 54.2, 128: 69.6 / 68.6, 192: 108.3 / 109.6.  At 128 MiB the
    // write-through stores are still draining when the next layer starts: 48 such layers back to back take 3.46 ms
    // against 3.41 ms with streaming stores, so the switch is at 96 MiB.
    rs.dx_cached = g_dx_cached >= 0 ? g_dx_cached != 0
                                    : (int64_t)B * T * D * (dt == LNPEGN_BF16 ? 2 : 4) <= ((int64_t)96 << 20);
    const hipError_t e = dt == LNPEGN_BF16 ? (saved ? launch_rows_bf16_saved(rs, a, rl) : launch_rows_bf16_recompute(rs, a, rl))
                                           : (saved ? launch_rows_f32_saved(rs, a, rl) : launch_rows_f32_recompute(rs, a, rl));
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return LNPEGN_EHIP;
    }
    if (defer) return LNPEGN_OK;   // lnpegn_reduce_deferred finishes the job

    // ---- the levels above the chunks (fixed-order sums) ----
    ReduceArgs ra{};
    ra.part = part;
    ra.grp = reinterpret_cast<float *>(ws + p.off_grp);
    ra.part_s = reinterpret_cast<double *>(ws + p.off_part_s);
    ra.part_big = reinterpret_cast<double *>(ws + p.off_part_big);
    ra.dgamma = dgamma; ra.dbeta = dbeta;
    ra.pe_gamma_sq = pe_gamma_sq; ra.pe_beta_sq = pe_beta_sq;
    ra.big_sq = pegn ? big_sq : nullptr;
    ra.n_slots = (int)p.n_slots; ra.gs = p.gs; ra.G1 = p.G1; ra.n_ex = p.n_ex; ra.ex_gs = p.C; ra.D = D; ra.ntile = p.ntile;
    ra.accumulate = accumulate;
    ra.nslab = p.nslab; ra.slab = reinterpret_cast<double *>(ws + p.off_grp); ra.arrived = &a.head->arrived;
    if (p.one_pass)
        return launch(slab_quads(D) == 8 ? reduce_slab_kernel<8> : reduce_slab_kernel<4>, dim3((unsigned)p.nslab),
                      dim3(kSlabThreads), 0, s, ra) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
    if (launch(reduce_groups_kernel, dim3((unsigned)p.ntile, (unsigned)reduce_groups_count(ra)), dim3(kTile), 0, s, ra) != hipSuccess) return LNPEGN_EHIP;
    const bool need_scalars = p.n_ex > 0 || ra.big_sq != nullptr;
    if (p.G1 == 1 || (int64_t)p.G1 * D <= kSmallFinal) {
        if (p.G1 > 1 || need_scalars) {
            if (launch(reduce_final_small_kernel, dim3(1), dim3(1024), 0, s, ra) != hipSuccess) return LNPEGN_EHIP;
        }
    } else {
        if (launch(reduce_final_tiles_kernel, dim3((unsigned)p.ntile), dim3(kTile), 0, s, ra) != hipSuccess) return LNPEGN_EHIP;
        if (need_scalars) {
            if (launch(reduce_scalars_kernel, dim3(1), dim3(256), 0, s, ra) != hipSuccess) return LNPEGN_EHIP;
        }
    }
    return LNPEGN_OK;
}

// Streaming yardstick: every lane moves 4 x 16 bytes per array, one workgroup per 16 KiB.
template <int kMode>
__global__ __launch_bounds__(256) void stream_probe_kernel(const uint4 *a, const uint4 *b, uint4 *out,
                                                           int64_t nvec)
{
    const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    uint4 va[4], vb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t v = base + i * 256;
        if (v < nvec) {
            va[i] = a[v];
            if (kMode == 1) vb[i] = b[v];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t v = base + i * 256;
        if (v < nvec) {
            uint4 o = va[i];
            if (kMode == 1) {
                o.x ^= vb[i].x; o.y ^= vb[i].y; o.z ^= vb[i].z; o.w ^= vb[i].w;
            }
            out[v] = o;
        }
    }
}

// The same with one vector per lane and array, streaming loads and stores, one workgroup per 4 KiB: the
// fastest plain streaming kernel found on this part (the workgroups are dealt out in address order and
// never loop, so the window of memory in use stays narrow).
__global__ __launch_bounds__(256) void stream_probe_oneshot_kernel(const uint4 *a, const uint4 *b, uint4 *out,
                                                                   int64_t nvec)
{
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v < nvec) {
        const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a) + v);
        const u32x4 y = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(b) + v);
        __builtin_nontemporal_store(x ^ y, reinterpret_cast<u32x4 *>(out) + v);
    }
}

template <typename T, bool kWriteY, bool kRagged>
hipError_t launch_fwd_vectors(FwdArgs a, hipStream_t s);

template <typename T, bool kWriteY>
hipError_t launch_fwd(FwdArgs a, bool vector_ok, hipStream_t s)
{
    constexpr int E = Vec<T>::kElems;
    const int D = a.D;
    const int64_t N = a.N;
    const uintptr_t any = reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.y) |
                          reinterpret_cast<uintptr_t>(a.gamma) | reinterpret_cast<uintptr_t>(a.beta);
    const bool element_ok = (any & (16 / E - 1)) == 0, fits = ceil_div(D, E) <= 64 * (16 / E) * 16;   // up to 16 waves share a row
    a.nvec = ceil_div(D, E);
    if (vector_ok && D % E == 0 && fits) return launch_fwd_vectors<T, kWriteY, false>(a, s);
    if (element_ok && D >= E && fits) return launch_fwd_vectors<T, kWriteY, true>(a, s);
    {
        const unsigned grid = (unsigned)(N < 4096 ? N : 4096);
        return launch(ln_fwd_generic_kernel<T, kWriteY>, dim3(grid), dim3(256), 0, s, a);
    }
}

template <typename T, bool kWriteY, bool kRagged>
hipError_t launch_fwd_vectors(FwdArgs a, hipStream_t s)
{
    constexpr int E = Vec<T>::kElems;
    const int64_t N = a.N;
    if (a.nvec <= 64 * (16 / E)) {
        const int vpt = ceil_div(a.nvec, 64);
        const int64_t want = (N + 3) / 4;
        const dim3 grid((unsigned)(want < 4096 ? want : 4096)), block(256);
        // bf16 rows ahead as soon as a wave has more than one.  us, without / with: D=768 N=16400 12.8 / 11.7, N=32768 20.5 / 19.0, D=1024
        // 24.8 / 23.7, D=256 N=65536 18.6 / 17.7; but N=8192 (one row a wave) 7.7 / 7.8, ragged rows (D=1001 N=32768) 26.3 / 27.7,
        // fp32 D=640 N=8192 9.3 / 9.8, D=512 N=32768 23.6 / 23.6.
        if constexpr (E == 8 && kWriteY && !kRagged) {
            if (N > 4 * 4096)
                return vpt == 1 ? launch(ln_fwd_kernel<T, 1, false, true, false, true>, grid, block, 0, s, a)
                                : launch(ln_fwd_kernel<T, 2, false, true, false, true>, grid, block, 0, s, a);
        }
        switch (vpt) {
            case 1: return launch(ln_fwd_kernel<T, 1, false, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 2: return launch(ln_fwd_kernel<T, 2, false, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 3: return launch(ln_fwd_kernel<T, 3, false, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 4: return launch(ln_fwd_kernel<T, 4, false, kWriteY, kRagged, false>, grid, block, 0, s, a);
            default: return hipErrorInvalidValue;
        }
    } else {
        const int waves = ceil_div(a.nvec, 64 * (16 / E));
        const int vpt = ceil_div(a.nvec, 64 * waves);
        // measured (B*T = 32768 rows, bf16): 16 resident waves per CU for rows of 2 and 4 waves (D=2048: 47.8 us
        // against 52.6 with twice as many; D=4096: 92.3 against 95.2), the full 32 for rows of 8 (D=8192: 181 against 190)
        const int64_t cap = waves <= 4 ? 4096 / waves : 4096;
        const dim3 grid((unsigned)(N < cap ? N : cap)), block(64 * waves);
        // bf16 rows of two waves: ahead where a workgroup has two to four.  us, without / with: D=2048 N=4096 8.9 / 7.8, N=8192
        // 14.3 / 13.6, D=1536 N=8192 12.1 / 11.3, D=1280 11.7 / 11.0; but D=2048 N=32768 46.6 / 48.6, three waves (D=3072 N=8192)
        // 20.3 / 21.0, four (D=4096 N=16384) 46.6 / 48.3, and fp32 D=2048 N=8192 24.1 / 25.3.
        if constexpr (E == 8 && kWriteY && !kRagged) {
            if (waves == 2 && N > cap && N <= 4 * cap) return launch(ln_fwd_kernel<T, 2, true, true, false, true>, grid, block, 0, s, a);
        }
        switch (vpt) {
            case 1: return launch(ln_fwd_kernel<T, 1, true, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 2: return launch(ln_fwd_kernel<T, 2, true, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 3: return launch(ln_fwd_kernel<T, 3, true, kWriteY, kRagged, false>, grid, block, 0, s, a);
            case 4: return launch(ln_fwd_kernel<T, 4, true, kWriteY, kRagged, false>, grid, block, 0, s, a);
            default: return hipErrorInvalidValue;
        }
    }
}

}  // namespace
}  // namespace lnpegn

using namespace lnpegn;

extern "C" {

size_t lnpegn_workspace_bytes(int B, int T, int D, lnpegn_dtype dt)
{
    if (!shape_ok(B, T, D) || !dtype_ok(dt)) return 0;
    size_t need = 0;
    for (int pegn = 0; pegn < 2; ++pegn)
        for (Access access : {kGenericAccess, kElementAccess, kVectorAccess}) {
            const size_t t = make_plan(B, T, D, dt, pegn != 0, access).total;
            if (t > need) need = t;
        }
    return need;
}

int lnpegn_plan_query(int B, int T, int D, lnpegn_dtype dt, int per_example, int aligned, int64_t *out, int n_out)
{
    if (!shape_ok(B, T, D) || !out || n_out < 0) return LNPEGN_EINVAL;
    if (!dtype_ok(dt)) return LNPEGN_EUNSUPPORTED;
    const Plan p = make_plan(B, T, D, dt, per_example != 0, aligned != 0 ? kVectorAccess : kElementAccess);
    const int64_t v[LNPEGN_PLAN_FIELDS] = {
        p.fast && !p.ragged ? 1 : 0, p.S, p.fast ? p.R : 1, p.vpt, p.C, p.n_slots, p.rows_per, p.stagger, p.xcd_chunks,
        (int64_t)p.lds_bytes, p.emit_pe ? 1 : 0, p.n_ex, p.G1, p.gs, (int64_t)p.total, p.Tp};
    for (int i = 0; i < n_out && i < LNPEGN_PLAN_FIELDS; ++i) out[i] = v[i];
    return LNPEGN_OK;
}

int lnpegn_last_hip_error(void) { return g_last_hip_error; }

const char *lnpegn_status_string(int status)
{
    switch (status) {
        case LNPEGN_OK: return "ok";
        case LNPEGN_EINVAL: return "invalid argument";
        case LNPEGN_EUNSUPPORTED: return "unsupported dtype";
        case LNPEGN_EWORKSPACE: return "workspace missing or too small";
        case LNPEGN_EHIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

int ln_fwd_stats(const void *x, float *mean, float *rstd, int B, int T, int D, lnpegn_dtype dt,
                 float eps, void *stream)
{
    if (!shape_ok(B, T, D) || !(eps >= 0.f)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt)) return LNPEGN_EUNSUPPORTED;
    if (!x || !mean || !rstd) return LNPEGN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FwdArgs a{};
    a.x = x; a.mean = mean; a.rstd = rstd; a.N = (int64_t)B * T; a.D = D; a.eps = eps;
    a.inv_D = 1.0f / (float)D;
    const hipError_t e = dt == LNPEGN_BF16 ? launch_fwd<bf16_t, false>(a, aligned16(x), s)
                                           : launch_fwd<float, false>(a, aligned16(x), s);
    return e == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int ln_fwd(const void *x, const void *gamma, const void *beta, void *y, float *mean, float *rstd, int B,
           int T, int D, lnpegn_dtype dt, lnpegn_dtype gamma_dt, float eps, void *stream)
{
    if (!shape_ok(B, T, D) || !(eps >= 0.f)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt) || !dtype_ok(gamma_dt)) return LNPEGN_EUNSUPPORTED;
    if (!x || !gamma || !beta || !y) return LNPEGN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FwdArgs a{};
    a.x = x; a.gamma = gamma; a.beta = beta; a.y = y; a.mean = mean; a.rstd = rstd;
    a.N = (int64_t)B * T; a.D = D; a.gamma_is_f32 = gamma_dt == LNPEGN_F32; a.eps = eps;
    a.inv_D = 1.0f / (float)D;
    const bool vec = aligned16(x) && aligned16(y) && aligned16(gamma) && aligned16(beta);
    const hipError_t e = dt == LNPEGN_BF16 ? launch_fwd<bf16_t, true>(a, vec, s)
                                           : launch_fwd<float, true>(a, vec, s);
    return e == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int ln_bwd(const void *x, const void *dy, const void *gamma, const float *mean, const float *rstd,
           void *dx, float *dgamma, float *dbeta, int B, int T, int D, lnpegn_dtype dt,
           lnpegn_dtype gamma_dt, float eps, void *workspace, size_t workspace_bytes, void *stream)
{
    return run_bwd(false, false, false, false, x, dy, gamma, mean, rstd, dx, dgamma, dbeta, nullptr, nullptr, nullptr, B, T,
                   D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int ln_bwd_pegn(const void *x, const void *dy, const void *gamma, const float *mean,
                const float *rstd, void *dx, float *dgamma, float *dbeta, float *pe_gamma_sq,
                float *pe_beta_sq, float *big_sq, int B, int T, int D, lnpegn_dtype dt,
                lnpegn_dtype gamma_dt, float eps, void *workspace, size_t workspace_bytes,
                void *stream)
{
    return run_bwd(true, false, false, false, x, dy, gamma, mean, rstd, dx, dgamma, dbeta, pe_gamma_sq, pe_beta_sq, big_sq,
                   B, T, D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int ln_bwd_pegn_static(const void *x, const void *dy, const void *gamma, const float *mean, const float *rstd,
                       void *dx, float *dgamma, float *dbeta, float *pe_gamma_sq, float *pe_beta_sq, float *big_sq,
                       int B, int T, int D, lnpegn_dtype dt, lnpegn_dtype gamma_dt, float eps, void *stream)
{
    // validate the shape against the fixed scratch before touching the device
    if (!shape_ok(B, T, D) || !(eps >= 0.f)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt) || !dtype_ok(gamma_dt)) return LNPEGN_EUNSUPPORTED;
    const Access access = access_of(x, dy, dx, gamma, dt);
    if (make_plan(B, T, D, dt, true, access).total > kStaticScratchBytes &&
        !(make_plan(B, T, D, dt, true, access).ragged && make_plan(B, T, D, dt, true, kGenericAccess).total <= kStaticScratchBytes))
        return LNPEGN_EWORKSPACE;
    void *ws = nullptr;
    const hipError_t e = static_scratch(&ws);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return LNPEGN_EHIP;
    }
    return run_bwd(true, false, false, false, x, dy, gamma, mean, rstd, dx, dgamma, dbeta, pe_gamma_sq, pe_beta_sq, big_sq,
                   B, T, D, dt, gamma_dt, eps, ws, kStaticScratchBytes, stream);
}

int ln_bwd_deferred(const void *x, const void *dy, const void *gamma, const float *mean,
                    const float *rstd, void *dx, float *dgamma, float *dbeta, int B, int T, int D,
                    lnpegn_dtype dt, lnpegn_dtype gamma_dt, float eps, void *workspace,
                    size_t workspace_bytes, void *stream)
{
    return run_bwd(false, true, false, false, x, dy, gamma, mean, rstd, dx, dgamma, dbeta, nullptr, nullptr, nullptr, B,
                   T, D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int ln_bwd_pegn_deferred(const void *x, const void *dy, const void *gamma, const float *mean,
                         const float *rstd, void *dx, float *dgamma, float *dbeta,
                         float *pe_gamma_sq, float *pe_beta_sq, float *big_sq, int B, int T, int D,
                         lnpegn_dtype dt, lnpegn_dtype gamma_dt, float eps, void *workspace,
                         size_t workspace_bytes, void *stream)
{
    return run_bwd(true, true, false, false, x, dy, gamma, mean, rstd, dx, dgamma, dbeta, pe_gamma_sq, pe_beta_sq,
                   big_sq, B, T, D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int ln_bwd_ex(const void *x, const void *dy, const void *gamma, const float *mean, const float *rstd,
              void *dx, float *dgamma, float *dbeta, float *pe_gamma_sq, float *pe_beta_sq, float *big_sq,
              int B, int T, int D, lnpegn_dtype dt, lnpegn_dtype gamma_dt, float eps, void *workspace,
              size_t workspace_bytes, unsigned flags, void *stream)
{
    if (flags & ~(unsigned)(LNPEGN_PER_EXAMPLE | LNPEGN_DEFER | LNPEGN_ACCUMULATE)) return LNPEGN_EINVAL;
    const bool pegn = (flags & LNPEGN_PER_EXAMPLE) != 0;
    return run_bwd(pegn, (flags & LNPEGN_DEFER) != 0, (flags & LNPEGN_ACCUMULATE) != 0, false, x, dy, gamma, mean,
                   rstd, dx, dgamma, dbeta, pegn ? pe_gamma_sq : nullptr, pegn ? pe_beta_sq : nullptr,
                   pegn ? big_sq : nullptr, B, T, D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int rms_fwd(const void *x, const void *gamma, void *y, float *rstd, int B, int T, int D, lnpegn_dtype dt,
            lnpegn_dtype gamma_dt, float eps, void *stream)
{
    if (!shape_ok(B, T, D) || !(eps >= 0.f)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt) || !dtype_ok(gamma_dt)) return LNPEGN_EUNSUPPORTED;
    if (!x || !gamma || !y) return LNPEGN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FwdArgs a{};
    a.x = x; a.gamma = gamma; a.beta = nullptr; a.y = y; a.mean = nullptr; a.rstd = rstd;
    a.N = (int64_t)B * T; a.D = D; a.gamma_is_f32 = gamma_dt == LNPEGN_F32; a.rms = 1; a.eps = eps;
    a.inv_D = 1.0f / (float)D;
    const bool vec = aligned16(x) && aligned16(y) && aligned16(gamma);
    const hipError_t e = dt == LNPEGN_BF16 ? launch_fwd<bf16_t, true>(a, vec, s)
                                           : launch_fwd<float, true>(a, vec, s);
    return e == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int rms_bwd_ex(const void *x, const void *dy, const void *gamma, const float *rstd, void *dx, float *dgamma,
               float *pe_gamma_sq, float *big_sq, int B, int T, int D, lnpegn_dtype dt, lnpegn_dtype gamma_dt,
               float eps, void *workspace, size_t workspace_bytes, unsigned flags, void *stream)
{
    if (flags & ~(unsigned)(LNPEGN_PER_EXAMPLE | LNPEGN_DEFER | LNPEGN_ACCUMULATE)) return LNPEGN_EINVAL;
    const bool pegn = (flags & LNPEGN_PER_EXAMPLE) != 0;
    return run_bwd(pegn, (flags & LNPEGN_DEFER) != 0, (flags & LNPEGN_ACCUMULATE) != 0, true, x, dy, gamma,
                   nullptr, rstd, dx, dgamma, nullptr, pegn ? pe_gamma_sq : nullptr, nullptr,
                   pegn ? big_sq : nullptr, B, T, D, dt, gamma_dt, eps, workspace, workspace_bytes, stream);
}

int lnpegn_reduce_deferred(void *const *workspaces, int n, int B, int T, int D, lnpegn_dtype dt,
                           void *stream)
{
    if (!workspaces || n <= 0 || !shape_ok(B, T, D)) return LNPEGN_EINVAL;
    if (!dtype_ok(dt)) return LNPEGN_EUNSUPPORTED;
    for (int i = 0; i < n; ++i)
        if (!workspaces[i] || reinterpret_cast<uintptr_t>(workspaces[i]) % kAlign) return LNPEGN_EINVAL;
    const Plan p = make_plan(B, T, D, dt, true, kVectorAccess);   // the offsets used depend on B and D only
    // Which form a layer takes was decided when its row kernel was launched (plain or per-example, aligned or not) and
    // stands in its header; a form that no layer of this shape can have taken is not launched.
    bool some_one = g_overridden, some_two = g_overridden;
    for (int pegn = 0; pegn < 2; ++pegn)
        for (Access access : {kGenericAccess, kElementAccess, kVectorAccess}) {
            const bool one = make_plan(B, T, D, dt, pegn != 0, access).one_pass;
            some_one = some_one || one;
            some_two = some_two || !one;
        }
    const int g1_max = B + kGroups;     // an example each, then the groups
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int first = 0; first < n; first += kBatchMax) {
        BatchArgs b{};
        b.n = n - first < kBatchMax ? n - first : kBatchMax;
        for (int i = 0; i < b.n; ++i) b.ws[i] = static_cast<char *>(workspaces[first + i]);
        b.D = D; b.ntile = p.ntile;
        b.off_grp = p.off_grp; b.off_part_s = p.off_part_s; b.off_part_big = p.off_part_big;
        b.off_part = p.off_part; b.nslab = p.nslab;
        const dim3 slabs((unsigned)p.nslab, (unsigned)b.n);
        if (!some_two) {
            if (launch(slab_quads(D) == 8 ? reduce_slab_batch_kernel<8> : reduce_slab_batch_kernel<4>, slabs, dim3(kSlabThreads), 0, s, b) != hipSuccess) return LNPEGN_EHIP;
            continue;
        }
        const bool mostly_one = p.one_pass;     // p is the plan that most calls have: few layers, if any, take the other form
        if (mostly_one) {
            const unsigned groups = (unsigned)(g1_max < kBatchGroups ? g1_max : kBatchGroups);
            if (launch(reduce_groups_few_batch_kernel, dim3((unsigned)p.ntile, groups, (unsigned)b.n), dim3(kTile), 0, s, b) != hipSuccess) return LNPEGN_EHIP;
            if (launch(slab_quads(D) == 8 ? reduce_last_batch_kernel<8> : reduce_last_batch_kernel<4>, slabs, dim3(1024), 0, s, b) != hipSuccess) return LNPEGN_EHIP;
            continue;
        }
        if (some_one && launch(slab_quads(D) == 8 ? reduce_slab_batch_kernel<8> : reduce_slab_batch_kernel<4>, slabs, dim3(kSlabThreads), 0, s, b) != hipSuccess)
            return LNPEGN_EHIP;
        if (launch(reduce_groups_batch_kernel, dim3((unsigned)p.ntile, (unsigned)g1_max, (unsigned)b.n), dim3(kTile), 0, s, b) != hipSuccess) return LNPEGN_EHIP;
        if (launch(reduce_final_batch_kernel, dim3((unsigned)b.n), dim3(1024), 0, s, b) != hipSuccess) return LNPEGN_EHIP;
    }
    return LNPEGN_OK;
}

int gns_estimate(const float *pe_sq, const float *big_sq, int n_groups, int B, float pe_scale,
                 float *out, void *stream)
{
    if (!pe_sq || !big_sq || !out || n_groups <= 0 || B <= 1) return LNPEGN_EINVAL;
    return launch(gns_estimate_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream),  pe_sq, big_sq, n_groups, B, pe_scale, out) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int gns_ema_update(double *state, const float *records, int n, double alpha, float *smoothed, void *stream)
{
    if (!state || !records || n <= 0 || !(alpha >= 0.0 && alpha < 1.0)) return LNPEGN_EINVAL;
    return launch(gns_ema_update_kernel, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),  state, records, n, alpha, smoothed) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int gns_offline(const float *records, int64_t n, float *out, void *stream)
{
    if (!records || !out || n < 2) return LNPEGN_EINVAL;
    return launch(gns_offline_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), records, n, out) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int gns_linear_accum_steps(int64_t tokens_seen, int64_t ramp_tokens, int accum_final)
{
    if (tokens_seen < 0 || ramp_tokens < 0 || accum_final < 1) return -LNPEGN_EINVAL;
    if (ramp_tokens == 0 || tokens_seen >= ramp_tokens) return accum_final;
    const __int128 num = (__int128)accum_final * tokens_seen;
    const int64_t a = (int64_t)((num + ramp_tokens - 1) / ramp_tokens);
    return a < 1 ? 1 : (a > accum_final ? accum_final : (int)a);
}

int lnpegn_set_tuning(int key, int value)
{
    if (value < 0) return LNPEGN_EINVAL;
    g_overridden = true;
    switch (key) {
        case 0:
            if (value > kMaxChunks) return LNPEGN_EINVAL;
            g_chunks_pegn = value;
            return LNPEGN_OK;
        case 1:
            if (value > kMaxChunks) return LNPEGN_EINVAL;
            g_chunks_plain = value;
            return LNPEGN_OK;
        case 2:
            if (value > 16) return LNPEGN_EINVAL;
            g_waves = value;
            return LNPEGN_OK;
        case 3:
            g_stagger = value == 0 ? -1 : value - 1;
            return LNPEGN_OK;
        case 4:
            if (value > 2) return LNPEGN_EINVAL;
            g_xcd = value - 1;          // 0 automatic, 1 never, 2 always
            return LNPEGN_OK;
        case 5:
            if (value > 4) return LNPEGN_EINVAL;
            g_vpt_max = value;
            return LNPEGN_OK;
        case 6:
            if (value < 1 || value > 65535) return LNPEGN_EINVAL;
            g_emb_run_blocks = value;
            return LNPEGN_OK;
        case 7:
            if (value > 2) return LNPEGN_EINVAL;
            g_dx_cached = value - 1;
            return LNPEGN_OK;
        case 8:
            if (value > 2) return LNPEGN_EINVAL;
            g_blocked = value - 1;
            return LNPEGN_OK;
        default: return LNPEGN_EINVAL;
    }
}

int lnpegn_stream_probe(const void *a, const void *b, void *out, size_t bytes, int mode, void *stream)
{
    if (!a || !out || (mode >= 1 && !b) || bytes == 0 || bytes % 16) return LNPEGN_EINVAL;
    if (mode < 0 || mode > 2) return LNPEGN_EINVAL;
    if (!aligned16(a) || !aligned16(out) || (mode >= 1 && !aligned16(b))) return LNPEGN_EINVAL;
    const int64_t nvec = (int64_t)(bytes / 16);
    const int64_t blocks = mode == 2 ? (nvec + 255) / 256 : (nvec + 1023) / 1024;
    if (blocks > INT32_MAX) return LNPEGN_EINVAL;
    hipEvent_t ev_start = g_ev_start, ev_stop = g_ev_stop;
    g_ev_start = g_ev_stop = nullptr;
    const uint4 *pa = static_cast<const uint4 *>(a), *pb = static_cast<const uint4 *>(b);
    uint4 *po = static_cast<uint4 *>(out);
    int64_t n = nvec;
    void *args[] = {&pa, &pb, &po, &n};
    const void *fn = mode == 0   ? reinterpret_cast<const void *>(stream_probe_kernel<0>)
                     : mode == 1 ? reinterpret_cast<const void *>(stream_probe_kernel<1>)
                                 : reinterpret_cast<const void *>(stream_probe_oneshot_kernel);
    const hipError_t e = hipExtLaunchKernel(fn, dim3((unsigned)blocks), dim3(256), args, 0,
                                            static_cast<hipStream_t>(stream), ev_start, ev_stop, 0);
    return e == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

int lnpegn_set_profile_events(void *start_event, void *stop_event)
{
    if ((start_event == nullptr) != (stop_event == nullptr)) return LNPEGN_EINVAL;
    g_ev_start = static_cast<hipEvent_t>(start_event);
    g_ev_stop = static_cast<hipEvent_t>(stop_event);
    return LNPEGN_OK;
}

}  // extern "C"
