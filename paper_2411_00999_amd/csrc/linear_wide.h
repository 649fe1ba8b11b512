// The matrix-core kernel with the larger tile, for bf16 operands whose rows are whole 16-byte chunks (included by
// linear_pegn.hip).
//
// The kernel with the smaller tile (256 x 128, eight waves of 64 x 64) is bound by LDS: a stage of 64 positions is read by
// its waves at 108 bytes a clock and written by its direct loads at 64, together the 1980 clocks that a stage takes, for 1024
// clocks of MFMAs; and by the lines that it fetches.  A wave tile of 128 x 96 reads 42 % less for the same products, and a
// tile of 256 x 192 fetches 22 % less; 192 accumulators for the example and 192 for the running total leave room for no more,
// at four waves with 512 registers each.  One wave to a SIMD has nobody to hide behind, so all that is not an MFMA goes out in
// their shadow, placed by hand: the next fragments' reads, the next loads and the scalar work for those (all of it
// between the blocks of MFMAs: B=16 T=2048 K=2048 L=8192 996 us, in their shadow 918).  A stage is 32 positions, 28 KiB, five deep; one
// barrier a stage.
// Measured, smaller / larger tile: that shape 1057 / 896 us (1228 TFLOP/s in a process of its own, 1130 late in a long one; the library's plain GEMM 1060), B=8 T=1024
// K=768 L=50304 684 / 548, B=64 T=1024 K=768 L=3072 357 / 272.
// What bounds it: the first shape takes 1.42-1.51 M clocks (smaller tile 1.98-2.11 M), 1.06 M of them MFMAs, at 1.4-1.7 GHz (1.5-1.9): the part
// limits its power while the matrix cores toggle.
#pragma once

namespace lnpegn {
namespace {

struct WideArgs {
    const char *x, *g;      // [B,T,K], [B,T,L] bf16, rows whole 16-byte chunks
    float *w;               // [K,L]
    float *tile_s;          // [B][tiles * kWaves]
    double *tile_big;       // parts of ||w'||^2: [full * kWaves], then [other tiles][kBlocks]
    int B, T, K, L;
    int tiles_k, tiles;     // tiles along k, in all
    int full;               // tiles that a workgroup finishes by itself
    int splits, per;        // the other tiles: splits of the examples, examples of one
    float *part;            // ... and their sums (more than one split): [split][other tile][wave][register][lane]
    int accumulate;
};

struct WideCfg {
    static constexpr int kWaves = 4, kMI = 4, kNI = 3;               // 2 x 2 waves of 128 x 96
    static constexpr int kTileK = 256, kTileL = 192;
    static constexpr int kStageT = 32, kBufs = 5;
    static constexpr int kXRow = kTileK * 2, kGRow = kTileL * 2;
    static constexpr int kXBytes = kStageT * kXRow, kStageBytes = kXBytes + kStageT * kGRow;
    static constexpr int kXLoads = kXBytes / 1024 / kWaves, kGLoads = (kStageBytes - kXBytes) / 1024 / kWaves;   // 4, 3
    static constexpr int kPart = kTileK * kTileL;                    // floats of a slot
    static constexpr int kBlocks = kWaves * kMI * kNI;               // 32 x 32 blocks of a tile
};

// One direct-to-LDS load through a buffer, hidden from the compiler like load_to_lds.
__device__ __forceinline__ void load_to_lds_buffer(uint32_t lds_addr, uint32_t voff, u32x4_t rsrc)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc)
                 : "memory");
}

typedef __attribute__((ext_vector_type(2))) uint32_t wide_u32x2_t;
struct WideFrags {
    wide_u32x2_t a[4][2], b[3][2];
};

// kAdd: the tiles that a workgroup finishes are added to w (the others by linear_wide_sum_kernel).  A kernel of its own: beside
// the other form its addresses took registers there (B=1 T=1822 K=640 L=2624, not added to, 38.7 -> 42.6 us).
template <bool kAdd>
__global__ __launch_bounds__(256, 1) void linear_wide_kernel(WideArgs a)
{
    using C = WideCfg;
    __shared__ __align__(1024) unsigned char lds[C::kBufs * C::kStageBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const int nst = (a.T + C::kStageT - 1) / C::kStageT, last_rows = a.T - (nst - 1) * C::kStageT;
    const int wm = wave & 1, wn = wave >> 1;

    // this workgroup's tile and examples: all of them, or a split's.  The workgroups of a split walk its examples side by side
    // and neighbours share an operand (runs of (tile, example) pairs without that, evenly long over all workgroups,
    // fetched so much more that B=16 T=2048 K=2048 L=8192 took 1041 us instead of 996).
    const bool whole = (int)blockIdx.x < a.full;
    const int rest = a.tiles - a.full, at = whole ? xcd_spread(blockIdx.x, a.full) : xcd_spread((int)blockIdx.x - a.full, rest * a.splits);
    const int split = whole ? 0 : at / rest, tile = whole ? at : a.full + at - split * rest;
    const int b_begin = whole ? 0 : split * a.per, b_end = whole ? a.B : min(a.B, b_begin + a.per);
    const bool direct = whole || a.splits == 1;
    const int widthx = a.K * 2, widthg = a.L * 2;

    // where a lane reads in a stage: see the transposing reads of the smaller tile.  Rows of g are 384 bytes: chunk ^ 4 on
    // every second pair of rows spreads four rows over all banks.
    const int s16 = lane & 15, grp = lane >> 4, rr = (grp >> 1) * 8 + (s16 >> 2);
    // (for g 64 bytes further per fragment, with the swizzle's sign by parity: fragments 0 and 2, and 1)
    const int low = (grp & 1) * 2 + ((s16 & 3) >> 1), flip = ((s16 >> 3) & 1) * (wn == 0 ? 64 : -64);
    uint32_t a_at[C::kMI], b_at[2];                                // in the stage being read
#pragma unroll
    for (int i = 0; i < C::kMI; ++i) a_at[i] = lds_base + rr * C::kXRow + (((wm * C::kMI + i) ^ (s16 >> 2)) * 4 + low) * 16 + (s16 & 1) * 8;
    b_at[0] = lds_base + C::kXBytes + rr * C::kGRow + (wn * C::kNI * 4 + low) * 16 + (s16 & 1) * 8 + flip;
    b_at[1] = b_at[0] - 2 * flip;

    const int k0 = tile % a.tiles_k * C::kTileK, l0 = tile / a.tiles_k * C::kTileL;
    const int nstages = (b_end - b_begin) * nst;

    // ---- loading
    uint32_t x_off[C::kXLoads], g_off[C::kGLoads];
#pragma unroll
    for (int n = 0; n < C::kXLoads; ++n) {
        const int r = (wave * C::kXLoads + n) * 2 + (lane >> 5), c = (lane & 31) ^ ((r & 3) << 2);
        x_off[n] = k0 + c * 8 < a.K ? (uint32_t)(r * widthx + c * 16) : 0x80000000u;
    }
#pragma unroll
    for (int n = 0; n < C::kGLoads; ++n) {
        const int at = (wave * C::kGLoads + n) * 64 + lane, r = at / 24, c = (at - r * 24) ^ (((r >> 1) & 1) << 2);
        g_off[n] = l0 + c * 8 < a.L ? (uint32_t)(r * widthg + c * 16) : 0x80000000u;
    }
    // A stage's loads go through two buffers, which end with its last row: base and size of the stage to load next, made
    // ready in parts of a few scalar instructions.  (Bases are below 2^48: what is added to a buffer's first two words never
    // reaches the stride.)
    auto buffer_of = [](const char *p, uint32_t bytes) {
        const uint64_t at = reinterpret_cast<uint64_t>(p);
        return u32x4_t{(uint32_t)at, (uint32_t)(at >> 32), bytes, 0x00020000u};
    };
    const uint32_t x_step = C::kStageT * widthx, x_rest = last_rows * widthx, g_step = C::kStageT * widthg, g_rest = last_rows * widthg;
    const uint32_t x_first = nst > 1 ? x_step : x_rest, g_first = nst > 1 ? g_step : g_rest;
    u32x4_t x_buf = buffer_of(a.x + ((int64_t)b_begin * a.T * a.K + k0) * 2, x_first - k0 * 2);
    u32x4_t g_buf = buffer_of(a.g + ((int64_t)b_begin * a.T * a.L + l0) * 2, g_first - l0 * 2);
    uint32_t x_bytes = x_first, g_bytes = g_first;             // of the stage that the buffers describe
    int load_stage = 1, left = nstages - 1;                    // the one behind it
    const uint32_t lds_x = lds_base + wave * (C::kXLoads * 1024), lds_end = lds_x + C::kBufs * C::kStageBytes;
    uint32_t load_to = lds_x;
    const uint32_t to_g = C::kXBytes - wave * ((C::kXLoads - C::kGLoads) * 1024);
    auto on = [](u32x4_t &buf, uint32_t bytes) {
        const uint64_t at = ((uint64_t)buf.y << 32 | buf.x) + bytes;
        buf.x = (uint32_t)at;
        buf.y = (uint32_t)(at >> 32);
    };
    bool last = false;
    auto prepare = [&](auto part_tag) {
        constexpr int part = decltype(part_tag)::value;
        if constexpr (part == 0) {
            last = load_stage >= nst - 1;                      // (nst 1: every stage is)
            load_stage = last ? 0 : load_stage + 1;
            on(x_buf, x_bytes);
        } else if constexpr (part == 1) {
            on(g_buf, g_bytes);
            x_bytes = last ? x_rest : x_step;
            g_bytes = last ? g_rest : g_step;
        } else if constexpr (part == 2) {
            x_buf.z = left > 0 ? x_bytes - k0 * 2 : 0u;
            g_buf.z = left > 0 ? g_bytes - l0 * 2 : 0u;
            --left;
        } else {
            load_to += C::kStageBytes;
            load_to = load_to == lds_end ? lds_x : load_to;
        }
    };
    auto load = [&](auto n_tag) {
        constexpr int n = decltype(n_tag)::value;
        if constexpr (n < C::kXLoads) load_to_lds_buffer(load_to + n * 1024, x_off[n], x_buf);
        else load_to_lds_buffer(load_to + to_g + (n - C::kXLoads) * 1024, g_off[n - C::kXLoads], g_buf);
    };
    auto fetch = [&]() {
        load(std::integral_constant<int, 0>{});
        load(std::integral_constant<int, 1>{});
        load(std::integral_constant<int, 2>{});
        load(std::integral_constant<int, 3>{});
        load(std::integral_constant<int, 4>{});
        load(std::integral_constant<int, 5>{});
        load(std::integral_constant<int, 6>{});
        prepare(std::integral_constant<int, 0>{});
        prepare(std::integral_constant<int, 1>{});
        prepare(std::integral_constant<int, 2>{});
        prepare(std::integral_constant<int, 3>{});
    };

    f32x16_t acc[C::kMI][C::kNI];
    float tot[C::kMI][C::kNI][16];
    auto keep = [](f32x16_t &v) { asm volatile("" : "+a"(v)); };
#pragma unroll
    for (int mi = 0; mi < C::kMI; ++mi)
#pragma unroll
        for (int ni = 0; ni < C::kNI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) tot[mi][ni][i] = 0.f;

    // reads of one fragment (two transposing reads), KK: first or second 16 positions of the stage
#define WIDE_READ(DST, ADDR, FURTHER, PITCH, KK)                                                                          \
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"                              \
                 : "=&v"(DST[0]), "=&v"(DST[1])                                                                            \
                 : "v"(ADDR), "n"((KK) * 16 * (PITCH) + (FURTHER)), "n"((KK) * 16 * (PITCH) + 4 * (PITCH) + (FURTHER))       \
                 : "memory")
    // ... and one direct load beside it (the reads keep its distance from the write of m0)
#define WIDE_READ_AND_LOAD(DST, ADDR, FURTHER, PITCH, KK, TO, ON, VOFF, BUF)                                              \
    asm volatile("s_add_u32 m0, %5, %6\n\tds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4\n\t"    \
                 "buffer_load_dwordx4 %7, %8, 0 offen lds"                                                                  \
                 : "=&v"(DST[0]), "=&v"(DST[1])                                                                            \
                 : "v"(ADDR), "n"((KK) * 16 * (PITCH) + (FURTHER)), "n"((KK) * 16 * (PITCH) + 4 * (PITCH) + (FURTHER)), "s"(TO),  \
                   "n"(ON), "v"(VOFF), "s"(BUF)                                                                             \
                 : "memory", "scc")
#define WIDE_KEEP(F)                                                                                                      \
    "+v"(F.a[0][0]), "+v"(F.a[0][1]), "+v"(F.a[1][0]), "+v"(F.a[1][1]), "+v"(F.a[2][0]), "+v"(F.a[2][1]), "+v"(F.a[3][0]), \
        "+v"(F.a[3][1]), "+v"(F.b[0][0]), "+v"(F.b[0][1]), "+v"(F.b[1][0]), "+v"(F.b[1][1]), "+v"(F.b[2][0]), "+v"(F.b[2][1])
    auto frag = [](const wide_u32x2_t (&v)[2]) { return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3)); };
    uint32_t read_at = 0;                                      // of the stage being read, in the ring
    // the MFMAs of one fragment set; in their shadow the reads of the next, and the next loads go out and are made ready.  A lone
    // wave issues an instruction every four clocks, eight to an MFMA: a stage is 108 of them (242 with every address made
    // where it is used: B=16 T=2048 K=2048 L=8192 918 us, so 896).
    auto block = [&](WideFrags &f, WideFrags &next, auto kk_tag, auto first_tag) {
        constexpr int kk = decltype(kk_tag)::value;
        constexpr bool kFirst = decltype(first_tag)::value;    // of an example: on top of zeros
        asm volatile("s_waitcnt lgkmcnt(0)" : WIDE_KEEP(f) : : "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < C::kMI; ++mi)
#pragma unroll
            for (int ni = 0; ni < C::kNI; ++ni) {
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(f.a[mi]), frag(f.b[ni]), kFirst ? f32x16_t{} : acc[mi][ni], 0, 0, 0);
                const int at = mi * C::kNI + ni;
                if constexpr (kk == 1) {
                    if (at == 0) WIDE_READ(next.b[0], b_at[0], 0, C::kGRow, kk);
                    if (at == 1) WIDE_READ(next.b[1], b_at[1], 64, C::kGRow, kk);
                    if (at == 2) WIDE_READ(next.b[2], b_at[0], 128, C::kGRow, kk);
                    if (at == 3) WIDE_READ(next.a[0], a_at[0], 0, C::kXRow, kk);
                    if (at == 4) WIDE_READ(next.a[1], a_at[1], 0, C::kXRow, kk);
                    if (at == 5) WIDE_READ(next.a[2], a_at[2], 0, C::kXRow, kk);
                    if (at == 6) WIDE_READ(next.a[3], a_at[3], 0, C::kXRow, kk);
                    if (at == 7) {                             // the read addresses go on to the next stage's
                        const uint32_t by = read_at == (C::kBufs - 1) * C::kStageBytes ? 0u - read_at : (uint32_t)C::kStageBytes;
                        read_at += by;
                        b_at[0] += by;
                        b_at[1] += by;
#pragma unroll
                        for (int i = 0; i < C::kMI; ++i) a_at[i] += by;
                    }
                } else {
                    const uint32_t load_g = load_to + to_g;
                    if (at == 0) WIDE_READ_AND_LOAD(next.b[0], b_at[0], 0, C::kGRow, kk, load_to, 0, x_off[0], x_buf);
                    if (at == 1) WIDE_READ_AND_LOAD(next.b[1], b_at[1], 64, C::kGRow, kk, load_to, 1024, x_off[1], x_buf);
                    if (at == 2) WIDE_READ_AND_LOAD(next.b[2], b_at[0], 128, C::kGRow, kk, load_to, 2048, x_off[2], x_buf);
                    if (at == 3) WIDE_READ_AND_LOAD(next.a[0], a_at[0], 0, C::kXRow, kk, load_to, 3072, x_off[3], x_buf);
                    if (at == 4) WIDE_READ_AND_LOAD(next.a[1], a_at[1], 0, C::kXRow, kk, load_g, 0, g_off[0], g_buf);
                    if (at == 5) WIDE_READ_AND_LOAD(next.a[2], a_at[2], 0, C::kXRow, kk, load_g, 1024, g_off[1], g_buf);
                    if (at == 6) WIDE_READ_AND_LOAD(next.a[3], a_at[3], 0, C::kXRow, kk, load_g, 2048, g_off[2], g_buf);
                    if (at == 7) prepare(std::integral_constant<int, 0>{});
                    if (at == 8) prepare(std::integral_constant<int, 1>{});
                    if (at == 9) prepare(std::integral_constant<int, 2>{});
                    if (at == 10) prepare(std::integral_constant<int, 3>{});
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    using First = std::integral_constant<int, 0>;
    using Second = std::integral_constant<int, 1>;
    WideFrags f0, f1;
    fetch();
    fetch();
    fetch();
    fetch();
    asm volatile("s_waitcnt vmcnt(21)\n\ts_barrier" ::: "memory");
    WIDE_READ(f0.b[0], b_at[0], 0, C::kGRow, 0);
    WIDE_READ(f0.b[1], b_at[1], 64, C::kGRow, 0);
    WIDE_READ(f0.b[2], b_at[0], 128, C::kGRow, 0);
#pragma unroll
    for (int i = 0; i < C::kMI; ++i) WIDE_READ(f0.a[i], a_at[i], 0, C::kXRow, 0);
    for (int b = b_begin; b < b_end; ++b) {
        auto stage = [&](auto first_tag) {
            block(f0, f1, Second{}, first_tag);
            // the next stage has landed here, and everywhere; the buffer before this stage's has been read
            asm volatile("s_waitcnt vmcnt(14)\n\ts_barrier" ::: "memory");
            block(f1, f0, First{}, std::false_type{});
#pragma unroll
            for (int t = 0; t < C::kMI * C::kNI; ++t) keep(acc[t / C::kNI][t % C::kNI]);
        };
        stage(std::true_type{});
        for (int st = 1; st < nst; ++st) stage(std::false_type{});
        // example boundary: the wave's part of the squared norm, and the tile into the total.  A tile at a time: all 384
        // accumulators are never in vector registers together (the empty statements say which file a value lives in:
        // the example's among the accumulation registers, the total's not).  The next fragments, read in the shadow of the
        // MFMAs, have arrived by now; waited for all the same, since here is where they would be moved if registers ran short.
        asm volatile("s_waitcnt lgkmcnt(0)" : WIDE_KEEP(f0) : : "memory");
        // Columns beyond the matrix are zeros times x, no number where that is infinite: a lane's part of them is left out.
        float ssq = 0.f;
#pragma unroll
        for (int ni = 0; ni < C::kNI; ++ni) {
            float column = 0.f;
#pragma unroll
            for (int mi = 0; mi < C::kMI; ++mi) {
                keep(acc[mi][ni]);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float v = acc[mi][ni][i];
                    column = fmaf(v, v, column);
                    tot[mi][ni][i] += v;
                    asm volatile("" : "+v"(tot[mi][ni][i]));       // here, not after the branch below
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            ssq += l0 + (wn * C::kNI + ni) * 32 + (lane & 31) < a.L ? column : 0.f;
        }
        const float sum = wave_sum(ssq);
        if (lane == 0) a.tile_s[((int64_t)b * a.tiles + tile) * C::kWaves + wave] = sum;
    }
    // no load may reach LDS after the workgroup has left it, no read be under way when its registers are used again
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : WIDE_KEEP(f0) : : "memory");

    // ---- write the total
    if (direct) {
        double bsq = 0.0;
        // (K and L are multiples of 8: the eight rows that a wave holds in four registers are in the matrix or are not.  With a branch
        // for every output the edges were 5400 instructions that a wave runs once: B=1 T=1822 K=640 L=2624 38.7 us, so 34.4.)
        // What is added to is loaded some blocks of 32 x 32 ahead (a load beside each addition, which every store then
        // waits for: that shape 89 us, so 36.5; B=4 T=97 K=7360 L=11520 730, so 221).
        constexpr int kTiles = C::kMI * C::kNI, kAhead = 4;
        auto row = [&](int t, int i) { return (wm * C::kMI + t / C::kNI) * 32 + (i >> 2) * 8 + (i & 3); };
        auto column = [&](int t) { return (wn * C::kNI + t % C::kNI) * 32; };
        float *const at_lane = a.w + ((int64_t)(k0 + (lane >> 5) * 4) * a.L + l0 + (lane & 31));
        auto each = [&](int t, auto body) __attribute__((always_inline)) {
            if (l0 + column(t) + (lane & 31) < a.L) {
#pragma unroll
                for (int q = 0; q < 16; q += 4)
                    if (k0 + row(t, q) < a.K) {
#pragma unroll
                        for (int i = q; i < q + 4; ++i) body(i, at_lane + ((int64_t)row(t, i) * a.L + column(t)));
                    }
            }
        };
        float old[kAhead][16];
        auto fetch_old = [&](int t) __attribute__((always_inline)) {  // (without branches; from inside the matrix where the block is not)
            if constexpr (kAdd) {
                const float *const from = a.w + ((int64_t)((lane >> 5) * 4) * a.L + min(l0 + column(t) + (lane & 31), a.L - 1));
#pragma unroll
                for (int i = 0; i < 16; ++i) old[t % kAhead][i] = from[(int64_t)(min(k0 + row(t, i & 12), a.K - 8) + (i & 3)) * a.L];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
#pragma unroll
        for (int t = 0; t < kAhead - 1; ++t) fetch_old(t);
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            if (t + kAhead - 1 < kTiles) fetch_old(t + kAhead - 1);
            each(t, [&](int i, float *p) {
                float v = tot[t / C::kNI][t % C::kNI][i];
                if constexpr (kAdd) v += old[t % kAhead][i];
                *p = v;
                bsq += (double)v * (double)v;
            });
            if constexpr (kAdd) __builtin_amdgcn_sched_barrier(0);
        }
        bsq = wave_sum_f64(bsq);
        if (tile < a.full) {
            if (lane == 0) a.tile_big[tile * C::kWaves + wave] = bsq;
        } else if (lane < C::kMI * C::kNI) {
            a.tile_big[a.full * C::kWaves + (tile - a.full) * C::kBlocks + wave * (C::kMI * C::kNI) + lane] = lane == 0 ? bsq : 0.0;
        }
    } else {
        // (the blocks of 32 x 32 that reach into the matrix: of K=8 L=1920 an eighth of 192 KiB)
        float *slot = a.part + (int64_t)at * C::kPart + wave * (C::kPart / C::kWaves) + lane;
#pragma unroll
        for (int mi = 0; mi < C::kMI; ++mi)
#pragma unroll
            for (int ni = 0; ni < C::kNI; ++ni)
                if (k0 + (wm * C::kMI + mi) * 32 < a.K && l0 + (wn * C::kNI + ni) * 32 < a.L) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) slot[((mi * C::kNI + ni) * 16 + i) * 64] = tot[mi][ni][i];
                }
    }
#undef WIDE_READ
#undef WIDE_READ_AND_LOAD
#undef WIDE_KEEP
}

// The tiles that several workgroups share: w = (accumulate ? w : 0) + the splits' sums, in order, and the parts of
// ||w'||^2.  grid (other tiles, kBlocks), 256 threads: four columns of a 32 x 32 block each.
__global__ __launch_bounds__(256) void linear_wide_sum_kernel(WideArgs a)
{
    using C = WideCfg;
    __shared__ double dslots[4];
    using Out = __attribute__((address_space(1))) u32x4_at4_t *;
    const int other = blockIdx.x, block = blockIdx.y, wave = block / (C::kMI * C::kNI), at = block % (C::kMI * C::kNI);
    const int tile = a.full + other, v = threadIdx.x * 4, i = v >> 6, ln = v & 63;
    const int k = tile % a.tiles_k * C::kTileK + ((wave & 1) * C::kMI + at / C::kNI) * 32 + (i >> 2) * 8 + (ln >> 5) * 4 + (i & 3);
    const int l = tile / a.tiles_k * C::kTileL + ((wave >> 1) * C::kNI + at % C::kNI) * 32 + (ln & 31);
    const float *slot = a.part + (int64_t)other * C::kPart + (int64_t)block * 1024 + v;
    const int64_t next = (int64_t)(a.tiles - a.full) * C::kPart;
    const bool inside = k < a.K && l < a.L;                        // (L is a multiple of 8)
    float *p = a.w + (int64_t)k * a.L + l;
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
    if (a.accumulate && inside) sum = __builtin_bit_cast(f32x4_t, (u32x4_t)*(Out)p);
    for (int j = 0; inside && j < a.splits; j += 4) {              // (blocks outside are not in the slots)
        f32x4_t u[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) u[n] = *reinterpret_cast<const f32x4_t *>(slot + min(j + n, a.splits - 1) * next);
#pragma unroll
        for (int n = 0; n < 4; ++n)
            if (j + n < a.splits) sum += u[n];
    }
    double q = 0.0;
    if (inside) {
        *(Out)p = __builtin_bit_cast(u32x4_t, sum);
        q = ((double)sum.x * sum.x + (double)sum.y * sum.y) + ((double)sum.z * sum.z + (double)sum.w * sum.w);
    }
    q = block_sum_f64(q, dslots);
    if (threadIdx.x == 0) a.tile_big[a.full * C::kWaves + other * C::kBlocks + block] = q;
}

}  // namespace
}  // namespace lnpegn
