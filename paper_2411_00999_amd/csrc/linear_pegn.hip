// Linear-layer simultaneous per-example gradient norms (Section 3, Algorithm 1) for gfx950:
//   w_b[k,l] = sum_t x[b,t,k] g[b,t,l]   (step 1; never leaves the chip)
//   s[b]     = sum_{k,l} w_b[k,l]^2      (step 2)
//   w'[k,l]  = sum_b w_b[k,l]            (step 3)
// One MFMA contraction per example with two accumulator sets per wave: the example's own tile, squared
// and folded into the running total at every example boundary.  The paper materialises [B,K,L] and
// pays its I/O (Section 3.1, Appendix E); here the only extra HBM traffic is B floats per tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/lnpegn.h"
#include "lnpegn_device.h"

namespace lnpegn {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// Workgroup tile: (WM*MI*32) (k) x (WN*NI*32) (l) outputs, 64 positions t per stage, WM x WN waves, each
// wave MI x NI MFMA tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16).
//
// A stage sits in LDS the way it sits in memory, [t][column]: 64 rows of x followed by 64 rows of g.
// It gets there by loads that write LDS directly (no registers in between), three stages deep: one
// being multiplied, one landed or landing, one just issued.  The MFMA operand of a lane is 8
// consecutive t of ONE column, i.e. a column of that layout; the transposing LDS read
// (ds_read_b64_tr_b16: 16 lanes read a 4 x 16 block as 4 rows, each lane receives one column of it)
// delivers exactly that, two reads per operand.  The four rows of such a block are a whole row pitch
// apart, which is a multiple of all banks, so the 16-byte chunks of row r are stored at chunk index
// c ^ 4*(r & 3); a direct-to-LDS load writes a wave's 64 chunks contiguously, so the swizzle is applied
// by choosing which chunk of memory each lane fetches.
constexpr int kBufs = 3, kMaxSplit = 64;

// kElem: bytes per element (2: bf16, 4: fp32).  A stage is 64 positions of bf16 or 32 of fp32: the same
// 48 KiB either way.
template <int WM, int WN, int MI, int NI, int kElem>
struct LinCfg {
    static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
    static constexpr int kTileK = WM * MI * 32, kTileL = WN * NI * 32;
    static constexpr int kStageT = 128 / kElem;
    static constexpr int kXRow = kTileK * kElem, kGRow = kTileL * kElem;  // bytes per LDS row
    static constexpr int kXBytes = kStageT * kXRow, kGBytes = kStageT * kGRow;
    static constexpr int kStageBytes = kXBytes + kGBytes;
    static constexpr int kXLoadsPerWave = kXBytes / 1024 / kWaves, kGLoadsPerWave = kGBytes / 1024 / kWaves;   // loads of 1 KiB
    static_assert(kXBytes % (1024 * kWaves) == 0 && kGBytes % (1024 * kWaves) == 0, "loads must divide evenly over the waves");
    static_assert(kXRow >= 256 && kGRow >= 256 && kXRow <= 1024 && kGRow <= 1024, "row of 16..64 chunks");
    static_assert(kBufs * kStageBytes <= 160 * 1024, "three stages must fit in LDS");
};
// 8 waves (two per SIMD, so one can issue MFMAs while the other waits for LDS), each 64 x 64: 256 x 128
// per workgroup.  Measured against 4 waves of 128 x 64 (one per SIMD, fewer LDS reads per MFMA): the
// lone wave cannot cover its own LDS latency and is 30 % slower.
typedef LinCfg<4, 2, 2, 2, 2> Cfg;       // tile shape and wave count are the same for both element types

struct LinArgs {
    const char *x;          // [B,T,K] bf16 or fp32
    const char *g;          // [B,T,L]
    float *out;             // nsplit == 1: w [K,L]; else partial totals [nsplit][K][L]
    float *tile_s;          // [B][ntiles*kWaves] per-wave parts of s[b]
    double *tile_big;       // [ntiles*kWaves] per-wave parts of ||w'||^2 (nsplit == 1 only)
    int B, T, K, L;
    int tiles_k, tiles_l, nsplit, b_per_split;
    int accumulate;         // nsplit == 1: add the total to what out holds
};

__device__ __forceinline__ int xcd_spread(int bid, int n)
{
    // Workgroups are handed to the 8 XCDs round-robin; give each XCD a contiguous run of logical
    // tiles (k fastest), so that workgroups sharing an operand share an L2.
    const int q = n >> 3, r = n & 7, xcd = bid & 7, loc = bid >> 3;
    return xcd * q + (xcd < r ? xcd : r) + loc;
}

// One direct-to-LDS load: every active lane moves 16 bytes from base + voff to LDS address
// lds_addr + 16*lane.  Written in assembly so that the compiler does not know of it: it would make the
// wave wait for the data before the next barrier, and the point is to wait two stages later.
__device__ __forceinline__ void load_to_lds(uint32_t lds_addr, uint32_t voff, const void *base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(base)
                 : "memory");
}

// The same for lanes that each have an address of their own.
__device__ __forceinline__ void load_to_lds_lane(uint32_t lds_addr, const void *lane_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_addr)
                 : "memory");
}

// The same as an instruction that the compiler counts, for kernels that load into registers besides: it waits for
// those by the number of loads behind them that it knows of, and with the direct loads hidden from it waits for
// most of them too.  (A buffer load: the global form it takes for one that completes out of order.)  A lane without
// data asks for an offset outside the buffer, and zeros are written.
constexpr int kTrackedBytes = 0x7ffffff0, kTrackedNone = INT32_MIN;
__device__ __forceinline__ void load_to_lds_tracked(uint32_t lds_addr, int voff, const void *base)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base, kTrackedBytes),
                                             (__attribute__((address_space(3))) void *)(uintptr_t)lds_addr, 16, voff, 0, 0, 0);
}

// What a lane reads whose chunk lies outside the matrix or behind the end of an example.
__device__ __constant__ uint32_t kZeroChunk[4] __attribute__((aligned(16))) = {0u, 0u, 0u, 0u};

// Sixteen bytes from an address that is only aligned to an element.
template <int kElem>
__device__ __forceinline__ u32x4_t load_chunk(const void *p)
{
    // (named as global memory: the waits behind a flat load are for everything under way)
    if constexpr (kElem == 2) return *(const __attribute__((address_space(1))) u32x4_at2_t *)p;
    else return *(const __attribute__((address_space(1))) u32x4_at4_t *)p;
}

// Ragged operands.  A direct-to-LDS load needs a 16-byte aligned address, so an operand whose rows do not all start
// on one (K or L no multiple of a chunk, or an unaligned pointer) takes another way: unaligned 16-byte loads into
// registers, written to the same places of the same LDS layout two stages later; everything behind the LDS is shared.
// (A copy of the operand with padded rows would take workspace of the operand's size and a pass over it.)  What
// bounds the ragged form is the time a load is given: with the registers written to LDS one stage after the load
// instead of two, and the aligned operand going the same way, B=8 T=1024 K=768 L=50257 took 1131 us against 861 us
// (735 TFLOP/s; the scalar kernel: 219 ms; L=50264, all direct: 703 us).
template <typename C, int WM, int WN, int MI, int NI, int kElem, bool kRaggedX, bool kRaggedG>
__device__ __forceinline__ void linear_pegn_body(const LinArgs &a)
{
    constexpr bool kF32 = kElem == 4, kRagged = kRaggedX || kRaggedG;
    constexpr int kStageT = C::kStageT, kPerChunk = 16 / kElem;       // elements per 16-byte chunk
    constexpr int kWaves = C::kWaves, kStageBytes = C::kStageBytes;
    constexpr int kXRow = C::kXRow, kGRow = C::kGRow, kXBytes = C::kXBytes;
    constexpr int kXLoads = C::kXLoadsPerWave, kGLoads = C::kGLoadsPerWave;
    __shared__ __align__(1024) unsigned char lds[kBufs * kStageBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: branches on it are scalar
    const int ntiles = a.tiles_k * a.tiles_l;
    const int tile = xcd_spread(blockIdx.x, ntiles);
    const int split = blockIdx.y;
    const int k0 = (tile % a.tiles_k) * C::kTileK, l0 = (tile / a.tiles_k) * C::kTileL;
    const int b_begin = split * a.b_per_split;
    const int b_end = b_begin + a.b_per_split < a.B ? b_begin + a.b_per_split : a.B;
    const int nst = (a.T + kStageT - 1) / kStageT;
    const int nstages = (b_end - b_begin) * nst;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;

    // ---- loading: a stage is loads of 1 KiB, kXLoads per wave for the rows of x and kGLoads for the rows of g.
    // Every wave issues the same number of loads at every stage and can count on that when it waits.  Behind the end
    // of an example lanes read a chunk of zeros; behind the edge of the matrix they load nothing (a load holds rows from
    // their first column on, so some lane of it always does) and their places in LDS are zeros from the start.
    // (An earlier form filled both with LDS stores and waited for all loads at every stage: an aligned layer with T no
    // multiple of a stage 1232 us against 909; zeros for the columns too: fp32 B=15 T=4096 K=64 L=1408 582 against 548.)
    const bool inside = k0 + C::kTileK <= a.K && l0 + C::kTileL <= a.L;
    const int last_rows = a.T - (nst - 1) * kStageT;           // rows of an example's last stage (64 if whole)
    // One operand: the stage to fetch next is tracked by a running pointer.  Rows are contiguous in memory, within
    // an example and from one example to the next, so a stage is 64 rows further unless it is the short last stage
    // of an example.
    struct Operand {
        const char *next;       // first element of this tile's columns, at the next stage to fetch
        const char *last;       // the last whole chunk of the tensor
        int stage;              // that stage's number within its example
        int left;               // stages still to fetch; behind the last, none or (ragged forms) rows of zeros
        int width, col0;        // columns in all, first column of the tile
    };
    Operand ox{a.x + ((int64_t)b_begin * a.T * a.K + k0) * kElem, a.x + (int64_t)a.B * a.T * a.K * kElem - 16, 0, nstages, a.K, k0};
    Operand og{a.g + ((int64_t)b_begin * a.T * a.L + l0) * kElem, a.g + (int64_t)a.B * a.T * a.L * kElem - 16, 0, nstages, a.L, l0};
    // Load n of this wave: the row and the chunk of memory that belong at this lane's LDS position.  fp32 operands
    // are read back one element per lane along a row, which needs no swizzle.
    auto row_of = [&](int load, int chunks, int ln) { return load * (64 / chunks) + ln / chunks; };
    auto chunk_of = [&](int row, int chunks, int ln) { return kF32 ? ln % chunks : (ln % chunks) ^ ((row & 3) << 2); };
    // The ragged forms have no register to spare (a spilled value read back in the loop waits for every load under
    // way: 4257 us for B=8 T=1024 K=769 L=50257 bf16): their addresses are made anew at every stage.
    auto own_lane = [&]() {
        int ln = lane;
        if constexpr (kRagged) asm volatile("" : "+v"(ln));
        return ln;
    };
    auto offset_of = [&](const Operand &o, int row, int chunk) { return (uint32_t)(((int64_t)row * o.width + chunk * kPerChunk) * kElem); };
    auto rows_at = [&](const Operand &o) { return o.left <= 0 ? 0 : o.stage == nst - 1 ? last_rows : kStageT; };
    auto advance = [&](Operand &o, int rows) {
        --o.left;
        o.next += (int64_t)rows * o.width * kElem;
        o.stage = o.stage == nst - 1 ? 0 : o.stage + 1;
    };
    constexpr bool kTracked = kRagged && !kF32;                // (fp32 reads its operands with loads the compiler knows of)
    // aligned rows: from memory to LDS
    auto fetch = [&](Operand &o, auto loads, auto chunks, uint32_t dst) {
        constexpr int kN = decltype(loads)::value, kChunks = decltype(chunks)::value;
        const int rows = rows_at(o);
        if (!kRagged && rows == 0) {                           // (chunks of zeros, one place for all to read: 1 us a call)
            --o.left;
            return;
        }
        const int ln = own_lane();
        auto to = [&](int n) { return dst + (wave * kN + n) * 1024; };
        if (!kTracked && inside && rows == kStageT) {
#pragma unroll
            for (int n = 0; n < kN; ++n) {
                const int r = row_of(wave * kN + n, kChunks, ln);
                load_to_lds(to(n), offset_of(o, r, chunk_of(r, kChunks, ln)), o.next);
            }
        } else {
#pragma unroll
            for (int n = 0; n < kN; ++n) {
                const int r = row_of(wave * kN + n, kChunks, ln), c = chunk_of(r, kChunks, ln);
                const bool column = o.col0 + c * kPerChunk < o.width;
                if constexpr (kTracked) load_to_lds_tracked(to(n), column && r < rows ? (int)offset_of(o, r, c) : kTrackedNone, o.next);
                else if (column) load_to_lds_lane(to(n), r < rows ? o.next + offset_of(o, r, c) : reinterpret_cast<const char *>(kZeroChunk));
            }
        }
        advance(o, rows);
    };
    // ragged rows: from memory to registers.  A chunk that begins inside its row may end in the next one: what it
    // brings along lands in columns behind the matrix, which count nowhere.  Only at the very end of a tensor is
    // there no next row; a chunk there is read from where it ends with the tensor (and shifted on its way to LDS).
    // One load each, whatever the place: with a branch around loads the compiler no longer knows how many are under
    // way, and waits for all of them.
    struct Fetched {
        const char *from;       // Operand::next
        int rows;
    };
    auto past_end = [&](const Operand &o, const Fetched &f, int r, int c) {  // bytes by which a chunk leaves its tensor
        const char *p = f.from + offset_of(o, r, c);
        return r < f.rows && o.col0 + c * kPerChunk < o.width && p > o.last ? (int)(p - o.last) : 0;
    };
    auto fetch_ragged = [&](Operand &o, auto loads, auto chunks, auto &regs, Fetched &f) {
        constexpr int kN = decltype(loads)::value, kChunks = decltype(chunks)::value;
        const int ln = own_lane();
        f = Fetched{o.next, rows_at(o)};
#pragma unroll
        for (int n = 0; n < kN; ++n) {
            const int r = row_of(wave * kN + n, kChunks, ln), c = chunk_of(r, kChunks, ln);
            const char *p = o.next + (o.col0 + c * kPerChunk < o.width ? offset_of(o, r, c) : offset_of(o, r, 0));
            p = p > o.last ? o.last : p;
            regs[n] = load_chunk<kElem>(r < f.rows ? p : reinterpret_cast<const char *>(kZeroChunk));
        }
        advance(o, f.rows);
    };
    // ... and from there to LDS; in assembly, because a store to LDS that the compiler knows of waits for every
    // direct load under way
    auto put = [&](const Operand &o, auto loads, auto chunks, auto &regs, const Fetched &f, uint32_t to) {
        constexpr int kN = decltype(loads)::value, kChunks = decltype(chunks)::value;
        if (f.rows > 0 && f.from + (int64_t)f.rows * o.width * kElem > o.last) {
            const int ln = own_lane();
#pragma unroll
            for (int n = 0; n < kN; ++n) {
                const int r = row_of(wave * kN + n, kChunks, ln);
                regs[n] = shift_down(regs[n], past_end(o, f, r, chunk_of(r, kChunks, ln)));
            }
        }
#pragma unroll
        for (int n = 0; n < kN; ++n) {
            const uint32_t at = to + (wave * kN + n) * 1024 + lane * 16;
            asm volatile("ds_write_b128 %0, %1" : : "v"(at), "v"(regs[n]) : "memory");
        }
    };
    using XLoads = std::integral_constant<int, kXLoads>;
    using GLoads = std::integral_constant<int, kGLoads>;
    using XChunks = std::integral_constant<int, kXRow / 16>;          // 16-byte chunks per row
    using GChunks = std::integral_constant<int, kGRow / 16>;
    constexpr int kSets = kRaggedX || kF32 ? 1 : 2;                    // stages under way in registers: as many as fit
    u32x4_t x_regs[kSets][kRaggedX ? kXLoads : 1], g_regs[kSets][kRaggedG ? kGLoads : 1];
    auto fetch_direct = [&](int buf) {                         // the aligned operands' next stage
        if constexpr (!kRaggedX) fetch(ox, XLoads{}, XChunks{}, lds_base + buf * kStageBytes);
        if constexpr (!kRaggedG) fetch(og, GLoads{}, GChunks{}, lds_base + buf * kStageBytes + kXBytes);
    };
    // The counts by which a wave waits for its direct loads hold only if those of a stage are issued before the register
    // loads that follow them here; both are loads that the compiler could order otherwise.
    auto in_order = [&]() { asm volatile("" ::: "memory"); };
    Fetched x_from[kSets], g_from[kSets];
    auto fetch_regs = [&](auto set) {                          // the ragged operands' next stage
        constexpr int s = decltype(set)::value;
        if constexpr (kRaggedX) fetch_ragged(ox, XLoads{}, XChunks{}, x_regs[s], x_from[s]);
        if constexpr (kRaggedG) fetch_ragged(og, GLoads{}, GChunks{}, g_regs[s], g_from[s]);
    };
    auto put_regs = [&](auto set, int buf) {
        constexpr int s = decltype(set)::value;
        if constexpr (kRaggedX) put(ox, XLoads{}, XChunks{}, x_regs[s], x_from[s], lds_base + buf * kStageBytes);
        if constexpr (kRaggedG) put(og, GLoads{}, GChunks{}, g_regs[s], g_from[s], lds_base + buf * kStageBytes + kXBytes);
    };

    // ---- multiplying: wave (wm, wn) owns outputs k0 + wm*MI*32 .. , l0 + wn*NI*32 .. .
    // For a transposing read, lane s of a 16-lane group reads row s/4 of the block, columns 4*(s%4) .. +3;
    // group g of the wave takes columns (g%2)*16 .. +15 of the 32 and positions (g/2)*8 .. +7 of the 16.
    const int wm = wave % WM, wn = wave / WM;
    const int s16 = lane & 15, grp = lane >> 4;
    const int rr = (grp >> 1) * 8 + (s16 >> 2);                // row within the 16 positions (first of two reads)
    uint32_t a_addr[MI], b_addr[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int q = (wm * MI + i) * 4 + (grp & 1) * 2 + ((s16 & 3) >> 1);
        a_addr[i] = rr * kXRow + ((q ^ ((s16 >> 2) << 2)) * 16) + (s16 & 1) * 8;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int q = (wn * NI + i) * 4 + (grp & 1) * 2 + ((s16 & 3) >> 1);
        b_addr[i] = kXBytes + rr * kGRow + ((q ^ ((s16 >> 2) << 2)) * 16) + (s16 & 1) * 8;
    }
    f32x16_t acc[MI][NI], tot[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc[mi][ni][i] = 0.f;
                tot[mi][ni][i] = 0.f;
            }
    // The transposing reads are written in assembly: the compiler's own selection of that instruction
    // takes no immediate offset (two VALU additions per read), and here the reads of the next 16
    // positions are issued, with immediate offsets off four per-stage addresses, before the MFMAs of the
    // current 16 start.  A block first waits for the reads issued by the block before it; the operands
    // those delivered are passed through it ("+v") so that no MFMA using them can be moved above the wait.
    static_assert(MI == 2 && NI == 2, "the read blocks below are written for 2 x 2 MFMA tiles per wave");
    static_assert(kF32 || 52 * (kXRow > kGRow ? kXRow : kGRow) < 65536, "immediate offsets of the reads");
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
    struct Frags {
        u32x2_t a0l, a0h, a1l, a1h, b0l, b0h, b1l, b1h;
    };
#define LIN_READS                                                                                              \
    "ds_read_b64_tr_b16 %0, %8 offset:%12\n\t"                                                                 \
    "ds_read_b64_tr_b16 %1, %8 offset:%13\n\t"                                                                 \
    "ds_read_b64_tr_b16 %2, %9 offset:%12\n\t"                                                                 \
    "ds_read_b64_tr_b16 %3, %9 offset:%13\n\t"                                                                 \
    "ds_read_b64_tr_b16 %4, %10 offset:%14\n\t"                                                                \
    "ds_read_b64_tr_b16 %5, %10 offset:%15\n\t"                                                                \
    "ds_read_b64_tr_b16 %6, %11 offset:%14\n\t"                                                                \
    "ds_read_b64_tr_b16 %7, %11 offset:%15"
#define LIN_ADDRS(KK)                                                                                          \
    "v"(pa0), "v"(pa1), "v"(pb0), "v"(pb1), "n"((KK) * 16 * kXRow), "n"((KK) * 16 * kXRow + 4 * kXRow),          \
        "n"((KK) * 16 * kGRow), "n"((KK) * 16 * kGRow + 4 * kGRow)
#define LIN_OUTS(F)                                                                                            \
    "=&v"(F.a0l), "=&v"(F.a0h), "=&v"(F.a1l), "=&v"(F.a1h), "=&v"(F.b0l), "=&v"(F.b0h), "=&v"(F.b1l), "=&v"(F.b1h)
#define LIN_KEEP(F)                                                                                            \
    "+v"(F.a0l), "+v"(F.a0h), "+v"(F.a1l), "+v"(F.a1h), "+v"(F.b0l), "+v"(F.b0h), "+v"(F.b1l), "+v"(F.b1h)
    auto mfmas = [&](const Frags &f) {
        const bf16x8_t fa[2] = {
            __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.a0l, f.a0h, 0, 1, 2, 3)),
            __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.a1l, f.a1h, 0, 1, 2, 3))};
        const bf16x8_t fb2[2] = {
            __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.b0l, f.b0h, 0, 1, 2, 3)),
            __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.b1l, f.b1h, 0, 1, 2, 3))};
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mi], fb2[ni], acc[mi][ni], 0, 0, 0);
    };
    // steps: groups of 16 positions that the stage holds (fewer than four at the end of an example)
    auto multiply_bf16 = [&](int buf, int steps, auto refill) {
        const uint32_t base = lds_base + buf * kStageBytes;
        const uint32_t pa0 = base + a_addr[0], pa1 = base + a_addr[1], pb0 = base + b_addr[0], pb1 = base + b_addr[1];
        Frags f0, f1;
        asm volatile(LIN_READS : LIN_OUTS(f0) : LIN_ADDRS(0) : "memory");
        asm volatile(LIN_READS : LIN_OUTS(f1) : LIN_ADDRS(1) : "memory");
        asm volatile("s_waitcnt lgkmcnt(8)" : LIN_KEEP(f0) : : "memory");
        mfmas(f0);
        asm volatile(LIN_READS : LIN_OUTS(f0) : LIN_ADDRS(2) : "memory");
        refill();                                              // later stages go out in the shadow of those MFMAs
        asm volatile("s_waitcnt lgkmcnt(8)" : LIN_KEEP(f1) : : "memory");
        if (steps > 1) mfmas(f1);
        asm volatile(LIN_READS : LIN_OUTS(f1) : LIN_ADDRS(3) : "memory");
        asm volatile("s_waitcnt lgkmcnt(8)" : LIN_KEEP(f0) : : "memory");
        if (steps > 2) mfmas(f0);
        asm volatile("s_waitcnt lgkmcnt(0)" : LIN_KEEP(f1) : : "memory");
        if (steps > 3) mfmas(f1);
    };
#undef LIN_READS
#undef LIN_ADDRS
#undef LIN_OUTS
#undef LIN_KEEP
    // fp32 operands (v_mfma_f32_32x32x2_f32: lane l holds row l%32 of A, column l%32 of B, position l/32 of
    // the two): one element per lane straight off a row of the stage, no transposition and no swizzle;
    // every read is one per-stage address plus an immediate.
    typedef __attribute__((address_space(3))) unsigned char lds_byte_t;
    typedef __attribute__((address_space(3))) float lds_float_t;
    uint32_t fa_addr[MI], fb_addr[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) fa_addr[i] = (lane >> 5) * kXRow + ((wm * MI + i) * 32 + (lane & 31)) * 4;
#pragma unroll
    for (int i = 0; i < NI; ++i) fb_addr[i] = kXBytes + (lane >> 5) * kGRow + ((wn * NI + i) * 32 + (lane & 31)) * 4;
    auto multiply_f32 = [&](int buf, auto refill) {
        const lds_byte_t *base = (const lds_byte_t *)lds + buf * kStageBytes;
        const lds_byte_t *pa[MI], *pb[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) pa[i] = base + fa_addr[i];
#pragma unroll
        for (int i = 0; i < NI; ++i) pb[i] = base + fb_addr[i];
        // The next pair's operands are read before the current pair's MFMAs start (left to itself the compiler reads them
        // after, and every pair waits for LDS: B=8 T=1024 K=768 L=2304 302 us against 285).
        float fa[2][MI], fb2[2][NI];
        auto read = [&](int ks) {
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[ks & 1][i] = *(const lds_float_t *)(pa[i] + ks * 2 * kXRow);
#pragma unroll
            for (int i = 0; i < NI; ++i) fb2[ks & 1][i] = *(const lds_float_t *)(pb[i] + ks * 2 * kGRow);
        };
        read(0);
#pragma unroll
        for (int ks = 0; ks < kStageT / 2; ++ks) {
            if (ks + 1 < kStageT / 2) read(ks + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[ks & 1][mi], fb2[ks & 1][ni], acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 1) refill();                             // later stages go out in the shadow of the MFMAs
        }
    };
    // outputs of a lane: rows (i/4)*8 + (lane/32)*4 + i%4, column lane%32 of each 32x32 tile
    auto out_k = [&](int mi, int i) { return k0 + (wm * MI + mi) * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3); };
    auto out_l = [&](int ni) { return l0 + (wn * NI + ni) * 32 + (lane & 31); };
    int cb = b_begin, cs = 0;                                  // the stage being multiplied
    auto multiply = [&](int buf, auto refill) {
        if constexpr (kF32) multiply_f32(buf, refill);
        else multiply_bf16(buf, ((cs == nst - 1 ? last_rows : kStageT) + 15) / 16, refill);
    };
    auto boundary = [&]() {
        if (++cs < nst) return;
        cs = 0;
        // example boundary: step 2 on this wave's part, then fold it into the total (step 3).  Outputs behind the
        // edge of the matrix are zero, or (ragged rows) made of whatever the rows' neighbours hold: not counted.
        float ssq = 0.f;
        int k_left = a.K, l_left = a.L;
        if constexpr (kRagged) asm volatile("" : "+s"(k_left), "+s"(l_left));   // 64 masks: made here, not kept in registers
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float v = acc[mi][ni][i];
                    const float counted = !kRagged || inside || (out_k(mi, i) < k_left && out_l(ni) < l_left) ? v : 0.f;
                    ssq = fmaf(counted, counted, ssq);
                    tot[mi][ni][i] += v;
                    acc[mi][ni][i] = 0.f;
                }
        ssq = wave_sum(ssq);
        if (lane == 0) a.tile_s[(int64_t)cb * (ntiles * kWaves) + tile * kWaves + wave] = ssq;
        ++cb;
    };

    // ---- pipeline: while stage st is multiplied the direct loads of stage st+2 go out, a ragged operand's registers
    // of stage st+1 (loaded one or two stages ago) are written to LDS, and the same registers receive the stage after
    // those under way.  Before it multiplies stage st a wave waits for its own direct loads of that stage (what it
    // issued later may still be under way); the barrier then says that every wave's part has landed and that stage
    // st-1 has been read by all, so its buffer can take stage st+2.
    constexpr int kDirect = (kRaggedX ? 0 : kXLoads) + (kRaggedG ? 0 : kGLoads);      // loads per wave and stage
    constexpr int kStaged = (kRaggedX ? kXLoads : 0) + (kRaggedG ? kGLoads : 0);
    static_assert(!(kRaggedX && !kRaggedG), "an x with ragged rows takes the kernel with both in registers");
    int cur = 0;                                               // buffer of stage st
    auto buffer = [&](int ahead) { return cur + ahead >= kBufs ? cur + ahead - kBufs : cur + ahead; };
    auto do_stage = [&](auto next_set) {
        // younger than the direct loads of stage st: those of st+1, the register loads of st+1 and st+2
        // (without ragged operands nothing is issued behind the last stage)
        if (!kRagged && ox.left < 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if constexpr (kDirect > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kDirect + kSets * kStaged) : "memory");
        if constexpr (kRagged) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // loads into registers stay under way
        else __syncthreads();
        // With ragged operands every stage issues the same loads, also where no stage is left (of zeros then): the
        // counts above, and the compiler's own for the registers, hold only if no path issues fewer.
        auto refill = [&]() {
            if constexpr (kRagged) put_regs(next_set, buffer(1));
            fetch_direct(buffer(2));
            if constexpr (kRagged) {
                in_order();
                fetch_regs(next_set);
            }
        };
        multiply(cur, refill);
        cur = buffer(1);
        boundary();
    };
    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, kSets - 1>;
    if constexpr (!kRagged) {
        if (!inside) {                                         // the places that no lane loads
            auto clear = [&](const Operand &o, int loads, int chunks, int at) {
                for (int i = wave * loads; i < (wave + 1) * loads; ++i)
                    if (o.col0 + chunk_of(row_of(i, chunks, lane), chunks, lane) * kPerChunk >= o.width)
                        for (int buf = 0; buf < kBufs; ++buf)
                            *reinterpret_cast<u32x4_t *>(lds + buf * kStageBytes + at + i * 1024 + lane * 16) = u32x4_t{0u, 0u, 0u, 0u};
            };
            clear(ox, kXLoads, kXRow / 16, 0);
            clear(og, kGLoads, kGRow / 16, kXBytes);
        }
    }
    fetch_direct(0);
    if constexpr (kRagged) {
        fetch_regs(Set0{});
        put_regs(Set0{}, 0);
    }
    if constexpr (kRagged) {
        fetch_regs(Set1{});
        in_order();
    }
    fetch_direct(1);
    if constexpr (kRagged) {
        in_order();
        if constexpr (kSets == 2) fetch_regs(Set0{});
        int st = 0;
        for (; st + 2 <= nstages; st += 2) {
            do_stage(Set1{});
            do_stage(Set0{});
        }
        if (st < nstages) do_stage(Set1{});
    } else {
        for (int st = 0; st < nstages; ++st) do_stage(Set0{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // no load may reach LDS after the workgroup has left it

    // ---- write the total
    float *out = a.out + (a.nsplit > 1 ? (int64_t)split * a.K * a.L : 0);
    double bsq = 0.0;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int l = out_l(ni);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int k = out_k(mi, i);
                if (k < a.K && l < a.L) {
                    float *p = out + (int64_t)k * a.L + l;
                    float v = tot[mi][ni][i];
                    if (a.accumulate && a.nsplit == 1) v += *p;
                    *p = v;
                    bsq += (double)v * (double)v;
                }
            }
        }
    if (a.nsplit == 1) {
        bsq = wave_sum_f64(bsq);
        if (lane == 0) a.tile_big[tile * kWaves + wave] = bsq;
    }
}

template <int kElem, bool kRaggedX, bool kRaggedG>
__global__ __launch_bounds__(Cfg::kThreads) void linear_pegn_kernel(LinArgs a)
{
    linear_pegn_body<LinCfg<4, 2, 2, 2, kElem>, 4, 2, 2, 2, kElem, kRaggedX, kRaggedG>(a);
}

}  // namespace
}  // namespace lnpegn
#include "linear_wide.h"
namespace lnpegn {
namespace {

// (ragged g beside aligned x: the rows of x are reached through 31-bit offsets)
template <int kElem>
hipError_t launch_linear(const LinArgs &a, bool ragged_x, bool ragged_g, hipStream_t st)
{
    const dim3 grid(a.tiles_k * a.tiles_l, a.nsplit), block(Cfg::kThreads);
    if (ragged_x || (ragged_g && a.K > (1 << 23))) return launch(linear_pegn_kernel<kElem, true, true>, grid, block, 0, st, a);
    if (ragged_g) return launch(linear_pegn_kernel<kElem, false, true>, grid, block, 0, st, a);
    return launch(linear_pegn_kernel<kElem, false, false>, grid, block, 0, st, a);
}

// Any shape, any alignment, fp32 or bf16: one thread per output (k,l), fp32 FMA over t, no MFMA.
// Correct, not fast; covers what the MFMA kernel does not take.
template <typename T>
__global__ __launch_bounds__(256) void linear_pegn_generic_kernel(const T *x, const T *g, float *w, float *blk_s,
                                                                  double *blk_big, int B, int Tn, int K, int L,
                                                                  int accumulate)
{
    __shared__ float slots[4];
    __shared__ double dslots[4];
    const int l = blockIdx.x * 16 + (threadIdx.x & 15), k = blockIdx.y * 16 + (threadIdx.x >> 4);
    const bool ok = k < K && l < L;
    const int blk = blockIdx.y * gridDim.x + blockIdx.x;
    float total = 0.f;
    for (int b = 0; b < B; ++b) {
        float acc = 0.f;
        if (ok) {
            const T *px = x + (int64_t)b * Tn * K + k, *pg = g + (int64_t)b * Tn * L + l;
            for (int t = 0; t < Tn; ++t)
                acc = fmaf(load_elem<T>(px, (int64_t)t * K), load_elem<T>(pg, (int64_t)t * L), acc);
        }
        total += acc;
        const float ssq = block_sum(acc * acc, slots);
        if (threadIdx.x == 0) blk_s[(int64_t)b * (gridDim.x * gridDim.y) + blk] = ssq;
    }
    double bsq = 0.0;
    if (ok) {
        float *p = w + (int64_t)k * L + l;
        if (accumulate) total += *p;
        *p = total;
        bsq = (double)total * (double)total;
    }
    bsq = block_sum_f64(bsq, dslots);
    if (threadIdx.x == 0) blk_big[blk] = bsq;
}

// w = (accumulate ? w : 0) + sum over splits, in split order; per-block parts of ||w||^2.  Four columns per thread, the loads of
// eight splits in flight (at any float: the rows of a split begin where they fall).  B=8 T=1024 K=768 L=2304, four splits:
// 10.9 us a column per thread, 7.0 so (call 55.8 -> 50.1; B=64 L=3072 369 -> 358).  Workgroups of 256 threads, or of one wave (`threads`,
// make_lin_plan).
constexpr int kSumEach = 4, kSumThreads = 256;
__global__ __launch_bounds__(kSumThreads) void linear_sum_splits_kernel(const float *part, float *w, double *blk_big,
                                                                        int64_t n, int nsplit, int accumulate)
{
    __shared__ double dslots[kSumThreads / 64];
    using In = const __attribute__((address_space(1))) u32x4_at4_t *;
    using Out = __attribute__((address_space(1))) u32x4_at4_t *;
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kSumEach;
    double bsq = 0.0;
    auto add = [&](auto load, auto store, auto &v) {
        v = accumulate ? load(w + i) : v;
        for (int s0 = 0; s0 < nsplit; s0 += 8) {
            std::remove_reference_t<decltype(v)> u[8];
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (s0 + s < nsplit) u[s] = load(part + (int64_t)(s0 + s) * n + i);
#pragma unroll
            for (int s = 0; s < 8; ++s)
                if (s0 + s < nsplit) v += u[s];
        }
        store(w + i, v);
    };
    if (i + kSumEach <= n) {
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        add([](const float *p) { return __builtin_bit_cast(f32x4_t, (u32x4_t)*(In)p); },
            [](float *p, f32x4_t v) { *(Out)p = __builtin_bit_cast(u32x4_t, v); }, v);
        bsq = ((double)v.x * v.x + (double)v.y * v.y) + ((double)v.z * v.z + (double)v.w * v.w);
    } else {
        for (int64_t left = i; left < n; ++left) {               // the last few columns
            float v = accumulate ? w[left] : 0.f;
            for (int s = 0; s < nsplit; ++s) v += part[(int64_t)s * n + left];
            w[left] = v;
            bsq += (double)v * (double)v;
        }
    }
    bsq = block_sum_f64(bsq, dslots);
    if (threadIdx.x == 0) blk_big[blockIdx.x] = bsq;
}

// s[b] = sum of its parts, big_sq = sum of the parts of ||w'||^2; fp64, in an order fixed by the launch
// shape alone (thread p % 1024 takes parts p, p + 1024, ...; then the fixed-order block sum).
// Workgroup b serves example b; workgroup B serves big_sq.
__global__ __launch_bounds__(1024) void linear_final_kernel(const float *part_s, int nparts, const double *part_big,
                                                            int64_t nbig, float *s, float *big_sq, int B)
{
    __shared__ double slots[16];
    const int b = blockIdx.x;
    double t = 0.0;
    if (b < B) {
        for (int p = threadIdx.x; p < nparts; p += 1024) t += (double)part_s[(int64_t)b * nparts + p];
        t = block_sum_f64(t, slots);
        if (threadIdx.x == 0) s[b] = (float)t;
    } else if (big_sq) {
        for (int64_t i = threadIdx.x; i < nbig; i += 1024) t += part_big[i];
        t = block_sum_f64(t, slots);
        if (threadIdx.x == 0) big_sq[0] = (float)t;
    }
}

struct LinPlan {
    bool mfma;             // matrix-core kernel
    bool ragged_x, ragged_g;   // rows of x, of g do not all start on 16-byte boundaries
    bool wide;             // ... with the larger tile
    int full;              // tiles of it that one workgroup finishes, whatever nsplit (of the others)
    int tiles_k, tiles_l, nsplit, b_per_split;
    int nparts;            // rows of the s parts
    int sum_threads;       // of a workgroup that adds the smaller tile's splits
    int64_t nbig;          // entries of the ||w'||^2 parts
    size_t off_s, off_big, off_part, bytes;
};
constexpr int kCUs = 256;
constexpr int kMaxSlots = 768;     // 192 KiB each

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// What make_lin_plan is told about the pointers.
struct LinAlign {
    bool x16, g16;         // on 16-byte boundaries
    bool element;          // on multiples of an element, both
};

// Which kernel: the faster one by the estimates below, that without the larger tile, or the one that is asked for.
enum LinKernel { kLinFaster, kLinNarrow, kLinMfma, kLinScalar };

// max_split: most workgroups that may share an output tile's examples (each but the first costs workspace).
LinPlan make_lin_plan(int B, int T, int K, int L, int dt, LinAlign align, LinKernel which = kLinFaster, int max_split = kMaxSplit)
{
    LinPlan p{};
    const int per_chunk = dt == LNPEGN_BF16 ? 8 : 4;          // elements per 16-byte vector
    p.ragged_x = K % per_chunk != 0 || !align.x16;
    p.ragged_g = L % per_chunk != 0 || !align.g16;
    // The matrix-core kernel takes every shape but ragged tensors of less than one chunk and rows so wide that the last of
    // a stage is beyond its offsets; those, and pointers that split an element, are left to the scalar kernel.
    const int64_t rows = (int64_t)B * T, tiles16 = (int64_t)((K + 15) / 16) * ((L + 15) / 16);
    const bool ragged = p.ragged_x || p.ragged_g;
    auto in_reach = [&](int width, bool own_ragged) {          // tracked loads: 31 bits of offset, all others 32
        const int esz = dt == LNPEGN_BF16 ? 2 : 4, stage = 128 / esz, last = (T < stage ? T : stage) - 1;
        const int64_t end = ((int64_t)last * width + Cfg::kTileK) * esz;
        return end <= (ragged && !own_ragged && dt == LNPEGN_BF16 ? (int64_t)kTrackedBytes : (int64_t)UINT32_MAX);
    };
    p.mfma = which != kLinScalar && in_reach(K, p.ragged_x) && in_reach(L, p.ragged_g) &&
             (!ragged || (align.element && rows * K >= per_chunk && rows * L >= per_chunk));
    if (p.mfma) {
        p.tiles_k = (K + Cfg::kTileK - 1) / Cfg::kTileK;
        p.tiles_l = (L + Cfg::kTileL - 1) / Cfg::kTileL;
        const int ntiles = p.tiles_k * p.tiles_l;
        // Split the examples when the output has fewer tiles than there are CUs, which hold one workgroup each: as the
        // time of the rounds of workgroups (1.1 us per bf16 stage, 3.5 per fp32 stage) and of adding the splits (a launch
        // and 128 KB written and read per tile and split) says.  At most as many splits as fill the CUs, which was the
        // rule before and ran four splits of 72 tiles, 288 workgroups, in two rounds.  us, that / this: bf16 B=8 T=1024 K=768 L=3072 87 / 70,
        // B=64 479 / 376, B=8 T=64 40 / 21, B=8 T=2048 K=2048 L=2560 262 / 221, B=5 T=512 K=768 L=2304 45 / 34, fp32 B=8
        // T=512 K=768 L=3072 284 / 223; unchanged where the splits fill one round (B=8 T=1024 K=768 L=2304 56).
        int most = (256 + ntiles - 1) / ntiles;
        if (most > B) most = B;
        if (most > max_split) most = max_split;
        const int stages = (T + Cfg::kStageT - 1) / Cfg::kStageT;
        const double stage_us = dt == LNPEGN_BF16 ? 1.1 : 3.5;
        double best = 0.0;
        for (int n = 1; n <= most; ++n) {
            const int per = (B + n - 1) / n, splits = (B + per - 1) / per, rounds = (ntiles * splits + 255) / 256;
            const double us = (double)rounds * per * stages * stage_us + (splits > 1 ? 2.0 + 0.045 * ntiles * splits : 0.0);
            if (n > 1 && us >= best) continue;
            best = us;
            p.b_per_split = per;
            p.nsplit = splits;
        }
        p.nparts = ntiles * Cfg::kWaves;
        // The splits are added by workgroups of one wave where those of 256 threads would be at most half as many as CUs.  us a
        // call, 256 threads / 64: B=10 T=268 K=64 L=2048 21.0 / 18.3, B=182 T=95 K=56 L=216 26.4 / 24.1; but, 143 workgroups of 256, B=11 T=81
        // K=2296 L=64 17.8 / 18.8, B=8 T=1024 K=768 L=2304 45.5 / 46.5, B=22 T=46 K=256 L=9216 32.1 / 34.0.  And where L is 128 or 2048, up to
        // 2^20 outputs: the product itself, the same code, then takes longer behind sums by larger workgroups (B=91 T=2 K=7808 L=128 34 / 40
        // of the call's 42.3 / 51.3; the sums and parts of a tile then meet in the caches of other XCDs): B=30 T=100 K=2688 L=128 27.1 /
        // 25.7, B=17 T=162 K=128 L=2048 24.6 / 21.1, B=3 T=146 K=512 L=2048 21.0 / 17.3; but K=768 L=2048 B=8 T=1024 44.0 / 45.2, and no
        // such difference at L of 512, 1024, 3072, 4096, 6144, 8192 (0.95 to 1.03).
        const int64_t outputs = (int64_t)K * L;
        p.sum_threads = outputs <= (int64_t)kCUs / 2 * kSumThreads * kSumEach || ((L == 128 || L == 2048) && outputs <= 1 << 20) ? 64 : kSumThreads;
        p.nbig = p.nsplit == 1 ? (int64_t)ntiles * Cfg::kWaves : (outputs + p.sum_threads * kSumEach - 1) / (p.sum_threads * kSumEach);
        // A few short ragged examples cost the matrix-core kernel its start and the scalar one little: the latter runs its
        // outputs side by side, an example and a position after the other.  us, matrix cores / scalar: bf16 B=1 T=8
        // K=257 L=300 14.3 / 6.5, T=100 16.0 / 15.8, T=300 20.5 / 36; B=3 T=8 K=1000 L=499 23 / 11; B=16 T=1 K=129 L=65 20 / 13,
        // T=8 20 / 24; fp32 B=1 T=300 K=129 L=65 58 / 37, B=3 T=100 33 / 37.
        const bool bf16 = dt == LNPEGN_BF16;
        const double mfma_us = (bf16 ? 12.4 : 13.6) + (double)((ntiles * p.nsplit + 255) / 256) * p.b_per_split * stages * (bf16 ? 1.3 : 8.0) +
                               4.5 * (p.b_per_split - 1) + (p.nsplit > 1 ? 3.0 + 0.045 * ntiles * p.nsplit : 0.0);
        const double position_us = ((tiles16 < 2 ? 0.065 : tiles16 < 16 ? 0.087 : 0.105) + 4e-6 * ((double)K + L) * (bf16 ? 2 : 4)) *
                                   (tiles16 > 2048 ? (double)tiles16 / 2048 : 1.0);
        const double scalar_us = 5.0 + B * (0.42 + 0.0002 * (double)tiles16 + position_us * T);
        if (ragged && which == kLinFaster && scalar_us < mfma_us) p.mfma = false;
    }
    if (!p.mfma) {
        p.tiles_k = (K + 15) / 16;
        p.tiles_l = (L + 15) / 16;
        p.nsplit = 1;
        p.b_per_split = B;
        p.nparts = p.tiles_k * p.tiles_l;
        p.nbig = p.nparts;
    }
    size_t slots = p.nsplit > 1 ? (size_t)p.nsplit * K * L * sizeof(float) : 0;
    // The larger tile of bf16: whole rounds of 256 workgroups finish a tile each; the examples of the other tiles are split over
    // workgroups.  Taken where it is the faster one by these estimates: the constants are those that fit 180 measured calls of
    // the smaller tile and 141 of this one (T 64 to 4096, K and L 64 to 8192), within 10 % nine times in ten.  They fit calls, not
    // kernels: of the 704 splits' sums of B=16 T=2048 K=2048 L=8192, 24.8 us by themselves, the price of a split bears 4.9 and the rounds
    // the rest (call 916 by the estimate, 890 to 910 measured; over 107 drawn calls of 400 to 768 sums 0.97 of it, of none 0.93).  us, smaller /
    // larger tile: B=16 T=2048 K=2048 L=8192 1047 / 933, L=2048 283 / 283, K=1280 L=5120 466 / 547; B=8 T=1024 K=768 L=50304 667 / 558,
    // L=3072 58.5 / 54.9, L=2304 46.7 / 51.0, K=4096 L=4096 267 / 258; B=64 T=1024 K=768 L=3072 351 / 281; B=32 T=512 K=1536 L=6144
    // 468 / 316; B=3 T=1000 K=1600 L=6400 112 / 71; B=9 T=4096 K=64 L=3840 155 / 82; B=16 T=512 K=1024 L=8192 143 / 159; B=64 T=128
    // K=1024 L=4096 98 / 119.
    if (p.mfma && !ragged && dt == LNPEGN_BF16 && which == kLinFaster &&
        (int64_t)WideCfg::kStageT * (K > L ? K : L) * 2 <= (int64_t)kTrackedBytes) {
        auto stages_of = [&](int each) { return (T + each - 1) / each; };
        // rounds of n workgroups; the last one quicker
        auto rounds = [](int64_t n, double least) {
            return n == 0 ? 0.0 : (double)((n - 1) / kCUs) + least + (1.0 - least) * (double)((n - 1) % kCUs + 1) / kCUs;
        };
        const int64_t narrow = (int64_t)p.tiles_k * p.tiles_l * p.nsplit;
        const bool edges = K % Cfg::kTileK != 0 || L % Cfg::kTileL != 0;       // (their loads are slower there)
        const double narrow_us = 4.1 + rounds(narrow, 0.885) * (p.b_per_split * ((edges ? 1.167 : 0.947) * stages_of(Cfg::kStageT) + 0.37) + 7.1) +
                                 (p.nsplit > 1 ? 2.1 + 0.044 * narrow : 0.0);
        const int tk = (K + WideCfg::kTileK - 1) / WideCfg::kTileK, tl = (L + WideCfg::kTileL - 1) / WideCfg::kTileL;
        const int64_t tiles = (int64_t)tk * tl, full = tiles / kCUs * kCUs, rest = tiles - full;
        const double pair_us = 0.599 * stages_of(WideCfg::kStageT) + 1.03;
        double us = 0.0;
        int splits = 1, per = B;
        // over every number of examples that a workgroup can be left with, by the fewest workgroups that leave it so (some
        // 2 sqrt(B) of them, 3 rounds at most); none to split where the tiles are whole rounds
        for (int each = B, m = 1;;) {
            const double t = 6.3 + (double)(full / kCUs) * (B * pair_us + 11.9) + rounds(rest * m, 0.61) * (each * pair_us + 11.9) +
                             (m > 1 ? 0.7 + 0.006 * rest * m : 0.0);
            if (m == 1 || t < us) {
                us = t;
                splits = m;
                per = each;
            }
            if (rest == 0 || each == 1) break;
            m = (B - 1) / (each - 1) + 1;
            each = (B - 1) / m + 1;
            if (rest * m > kMaxSlots) break;
        }
        if (us + 1.5 < 0.97 * narrow_us && per * stages_of(WideCfg::kStageT) >= 16) {
            p.wide = true;
            p.full = (int)full;
            p.tiles_k = tk;
            p.tiles_l = tl;
            p.nsplit = splits;
            p.b_per_split = per;
            p.nparts = (int)tiles * WideCfg::kWaves;
            p.nbig = full * WideCfg::kWaves + rest * WideCfg::kBlocks;
            slots = splits > 1 ? (size_t)(rest * splits) * WideCfg::kPart * sizeof(float) : 0;
        }
    }
    p.off_s = 0;
    p.off_big = align256(p.off_s + (size_t)p.nparts * B * sizeof(float));
    p.off_part = align256(p.off_big + (size_t)p.nbig * sizeof(double));
    p.bytes = p.off_part + slots;
    return p;
}

bool lin_shape_ok(int B, int T, int K, int L)
{
    return B > 0 && T > 0 && K > 0 && L > 0 && (int64_t)K * L <= ((int64_t)1 << 31);
}

}  // namespace
}  // namespace lnpegn

using namespace lnpegn;

extern "C" {

size_t linear_pegn_workspace_bytes(int B, int T, int K, int L, lnpegn_dtype dt)
{
    if (!lin_shape_ok(B, T, K, L) || (dt != LNPEGN_F32 && dt != LNPEGN_BF16)) return 0;
    // sized for either kernel, whatever the alignment of the pointers turns out to be
    size_t most = 0;
    for (int aligned = 0; aligned < 2; ++aligned)
        for (int element = aligned; element < 2; ++element) {
            const size_t n = make_lin_plan(B, T, K, L, dt, LinAlign{aligned != 0, aligned != 0, element != 0}).bytes;
            if (n > most) most = n;
        }
    return most;
}

int linear_pegn_plan_query(int B, int T, int K, int L, lnpegn_dtype dt, int aligned, int64_t *out, int n_out)
{
    if (!lin_shape_ok(B, T, K, L) || !out || n_out < 0) return LNPEGN_EINVAL;
    if (dt != LNPEGN_F32 && dt != LNPEGN_BF16) return LNPEGN_EUNSUPPORTED;
    const LinPlan p = make_lin_plan(B, T, K, L, dt, LinAlign{aligned != 0, aligned != 0, true});
    const int64_t v[LINEAR_PEGN_PLAN_FIELDS] = {p.wide ? 2 : p.mfma ? 1 : 0, (int64_t)p.tiles_k * p.tiles_l, p.full, p.nsplit, p.b_per_split,
                                                (int64_t)p.bytes};
    for (int i = 0; i < n_out && i < LINEAR_PEGN_PLAN_FIELDS; ++i) out[i] = v[i];
    return LNPEGN_OK;
}

int linear_pegn(const void *x, const void *g, float *w, float *s, float *big_sq, int B, int T, int K, int L,
                lnpegn_dtype dt, void *workspace, size_t workspace_bytes, unsigned flags, void *stream)
{
    if (!lin_shape_ok(B, T, K, L) || !x || !g || !w || !s || !workspace) return LNPEGN_EINVAL;
    if (flags & ~(unsigned)LNPEGN_ACCUMULATE) return LNPEGN_EINVAL;
    if (dt != LNPEGN_F32 && dt != LNPEGN_BF16) return LNPEGN_EUNSUPPORTED;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return LNPEGN_EINVAL;
    const uintptr_t px = reinterpret_cast<uintptr_t>(x), pg = reinterpret_cast<uintptr_t>(g), elem = dt == LNPEGN_BF16 ? 2 : 4;
    const LinAlign align{(px & 15u) == 0, (pg & 15u) == 0, ((px | pg) & (elem - 1)) == 0};
    LinPlan p = make_lin_plan(B, T, K, L, dt, align);
    // The larger tile may ask for more workspace than the smaller one, which is taken where it is not given.
    if (p.wide && workspace_bytes < p.bytes) p = make_lin_plan(B, T, K, L, dt, align, kLinNarrow);
    // Ragged rows run in less workspace too, down to what the scalar kernel asks for: without a split, or there.
    if (p.ragged_x || p.ragged_g) {
        if (workspace_bytes < p.bytes) p = make_lin_plan(B, T, K, L, dt, align, kLinMfma);
        if (workspace_bytes < p.bytes) p = make_lin_plan(B, T, K, L, dt, align, kLinMfma, 1);
        if (workspace_bytes < p.bytes) p = make_lin_plan(B, T, K, L, dt, align, kLinScalar);
    }
    if (workspace_bytes < p.bytes) return LNPEGN_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int accumulate = (flags & LNPEGN_ACCUMULATE) ? 1 : 0;
    char *ws = static_cast<char *>(workspace);
    float *part_s = reinterpret_cast<float *>(ws + p.off_s);
    double *part_big = reinterpret_cast<double *>(ws + p.off_big);
    float *part_w = reinterpret_cast<float *>(ws + p.off_part);
    if (p.wide) {
        WideArgs a{};
        a.x = static_cast<const char *>(x);
        a.g = static_cast<const char *>(g);
        a.w = w;
        a.tile_s = part_s;
        a.tile_big = part_big;
        a.part = part_w;
        a.B = B; a.T = T; a.K = K; a.L = L;
        a.tiles_k = p.tiles_k; a.tiles = p.tiles_k * p.tiles_l;
        a.full = p.full; a.splits = p.nsplit; a.per = p.b_per_split;
        a.accumulate = accumulate;
        if (launch(accumulate ? linear_wide_kernel<true> : linear_wide_kernel<false>, dim3(p.full + (a.tiles - p.full) * p.nsplit), dim3(64 * WideCfg::kWaves), 0, st, a) != hipSuccess) return LNPEGN_EHIP;
        if (p.nsplit > 1 && launch(linear_wide_sum_kernel, dim3(a.tiles - p.full, WideCfg::kBlocks), dim3(256), 0, st, a) != hipSuccess) return LNPEGN_EHIP;
    } else if (p.mfma) {
        LinArgs a{};
        a.x = static_cast<const char *>(x);
        a.g = static_cast<const char *>(g);
        a.out = p.nsplit > 1 ? part_w : w;
        a.tile_s = part_s;
        a.tile_big = part_big;
        a.B = B; a.T = T; a.K = K; a.L = L;
        a.tiles_k = p.tiles_k; a.tiles_l = p.tiles_l; a.nsplit = p.nsplit; a.b_per_split = p.b_per_split;
        a.accumulate = accumulate;
        const hipError_t e = dt == LNPEGN_BF16 ? launch_linear<2>(a, p.ragged_x, p.ragged_g, st)
                                               : launch_linear<4>(a, p.ragged_x, p.ragged_g, st);
        if (e != hipSuccess) return LNPEGN_EHIP;
        if (p.nsplit > 1) {
            const int64_t n = (int64_t)K * L;
            if (launch(linear_sum_splits_kernel, dim3((unsigned)p.nbig), dim3(p.sum_threads), 0, st, part_w, w, part_big, n, p.nsplit, accumulate) != hipSuccess) return LNPEGN_EHIP;
        }
    } else {
        const dim3 grid(p.tiles_l, p.tiles_k);
        const hipError_t e =
            dt == LNPEGN_BF16
                ? launch(linear_pegn_generic_kernel<bf16_t>, grid, dim3(256), 0, st, static_cast<const bf16_t *>(x),
                         static_cast<const bf16_t *>(g), w, part_s, part_big, B, T, K, L, accumulate)
                : launch(linear_pegn_generic_kernel<float>, grid, dim3(256), 0, st, static_cast<const float *>(x),
                         static_cast<const float *>(g), w, part_s, part_big, B, T, K, L, accumulate);
        if (e != hipSuccess) return LNPEGN_EHIP;
    }
    return launch(linear_final_kernel, dim3(B + 1), dim3(1024), 0, st, part_s, p.nparts, part_big, p.nbig, s, big_sq, B) == hipSuccess ? LNPEGN_OK : LNPEGN_EHIP;
}

}  // extern "C"
