// gfx950 kernel: the collapsed update with the Gram matrix of the gradient rows
// formed on the matrix cores.
//
// The per-group norms of a long update stream are quadratic forms in the Gram
// matrix Gamma_ab = sum_j g_a[j] g_b[j] (gradient-norm signal, Sections 4.3.1
// and 7 of the paper).  Gamma is a genuine dense contraction -- W x P times
// P x W -- and the only one on this path; everything else stays element-wise
// vector code.  On the vector ALUs Gamma costs W(W+1)/2 accumulator registers
// per thread, which caps the route at 16 rows and leaves one wave per SIMD;
// here it costs 4 (16-row tile) or 16 (32-row tile) accumulator registers per
// lane, so up to 32 rows fit in one pass.
//
// Data flow per wave and tile: the lanes hold, as in the other kernels, 4
// consecutive elements of every row (coalesced 16/8-byte loads) and apply the
// element-wise update from registers.  For the matrix cores the same values
// are needed "the other way round" (lane = row): they are staged through a
// wave-private LDS panel  T[row][element], 8 bytes per lane and row at a
// time, and read back 16 bytes at a time as  lane (i, t) <- T[i][part t].
#include "star_device.h"

#include <type_traits>

namespace star {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Matrix tiles.  "Row" is a gradient row (a worker), "slot" a group of lanes that feeds one part of
// the reduction dimension; lane l feeds row l % N and slot l / N.
//   fp32 rows, N=16: v_mfma_f32_16x16x4_f32,   1 element per lane, 4 slots
//   fp32 rows, 17 to 24: pairs of row groups of four by v_mfma_f32_4x4x1_16b_f32 (see kQuads in the kernel);
//   fp32 rows, 25 to 32: three 16x16 blocks by v_mfma_f32_16x16x4_f32 with A and B from the two halves of
//                    the rows (see kBlocks in the kernel); the 32x32x2 instruction is not used
//   bf16 rows, N=16: v_mfma_f32_16x16x32_bf16, 8 elements per lane, 4 slots
//   bf16 rows, N=32: v_mfma_f32_32x32x16_bf16, 8 elements per lane, 2 slots
// (products of two bf16 values are exact in fp32, so the bf16 instructions lose nothing; they
// run at 8 to 16 times the fp32 rate).  Result register r of lane l is
//   N=16: D[4*(l/16) + r][l%16],     N=32: D[(r%4) + 4*(l/32) + 8*(r/4)][l%32].
// Operands A and B of  D += A * B  are the same register: whatever order the instruction gives
// the reduction dimension inside a lane, it is the same for A and for B, so D accumulates
// sum_e g_i[e] g_j[e] = Gamma_ij.
template <bool WIDE>
struct GramTile;
template <>
struct GramTile<false> {
    static constexpr int N = 16, SLOTS = 4, REGS = 4;
    typedef f32x4 acc_t;
    static __device__ __forceinline__ acc_t mma(float x, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(x, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ acc_t mma(bf16x8 x, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int lane_of(int i, int j) { return 16 * (i / 4) + j; }
    static __device__ __forceinline__ int reg_of(int i) { return i % 4; }
};
template <>
struct GramTile<true> {
    static constexpr int N = 32, SLOTS = 2, REGS = 16;
    typedef f32x16 acc_t;
    static __device__ __forceinline__ acc_t mma(float x, acc_t c) {   // not reached: fp32 rows go by blocks
        return __builtin_amdgcn_mfma_f32_32x32x2f32(x, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ acc_t mma(bf16x8 x, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int lane_of(int i, int j) { return 32 * ((i % 8) / 4) + j; }
    static __device__ __forceinline__ int reg_of(int i) { return 4 * (i / 8) + (i % 4); }
};

// One row of the LDS panel holds 512 bytes of elements (128 fp32 or 256 bf16) and 16 bytes of
// padding: 16 lanes that read 16 bytes each from 16 consecutive rows at the same offset then
// touch every bank exactly once.
constexpr int kPanelRowBytes = 512 + 16;
// Row groups of four (kQuads): 16 lanes read 16 bytes each from 4 consecutive rows, 4 neighbouring places of each.
constexpr int kQuadRowBytes = 512 + 64;
// Which launches form the matrix from row groups of four, see the kernel.
constexpr bool quad_groups(bool bf16_rows, int W) { return !bf16_rows && W > 16 && W <= 24; }

// LDS of a workgroup without bursts, and the tiles of results that it holds beside that.
constexpr int panel_lds(bool bf16_rows, int W) {
    const bool quads = quad_groups(bf16_rows, W);
    const int pairs = (W / 4) * (W / 4 + 1) / 2;
    const int panel = kBlock / 64 * (quads ? W * kQuadRowBytes : (W > 16 ? 32 : 16) * kPanelRowBytes);
    return panel + (quads ? kBlock / 64 * ((pairs + 1) / 2) * 64 * 8 : 8);
}
constexpr int burst_tiles_beside_panel(bool bf16_rows, int W) { return burst_tiles(panel_lds(bf16_rows, W)); }

// What an update keeps on a compute unit: up to two workgroups (Shared), or one, with a tile of look-ahead, which writes as it goes (Alone) or
// keeps its results in LDS and writes them in bursts (Bursts, see Burst; two workgroups with half the room each, 16 fp32 / bf16 rows, 110 /
// 150 M elements: 1 487 / 1 227 us against 1 406 / 1 128).
//
// A unit's only workgroup has one wave per SIMD, which issues an instruction every four cycles at best and hides nothing behind another
// wave.  At the full clock of 2.4 GHz that is covered by the memory's time; but from 3 to 15 ms after a pause this card runs at 1.5 GHz, and
// there such a wave's instructions are what a tile takes (16 bf16 rows: 3 100 of 3 740 cycles).  So these forms (the `kAlone` path) hold two
// tiles in two sets of registers that take turns, instead of moving one to the other (104 moves a tile with 16 bf16 rows, 200 with fp32 rows), keep
// the map's coefficients in vector registers (else the row pointers do not fit into the scalar ones and are fetched back lane by lane), and
// mix the update into the matrix instructions, whose operands are read from LDS a step ahead.  250 ms idle, then four calls, us: 16 bf16
// rows, 340 M elements 11 395 -> 10 740 (two workgroups writing as they go 10 779), 12 bf16 rows, 200 M 5 690 -> 5 377 (5 303), 32 bf16 rows,
// 80 M 5 001 -> 4 795 (5 299), 16 fp32 rows, 110 M 6 732 -> 6 310 (6 631), 20 fp32 rows, 60 M 4 760 -> 4 395 (4 331).  Back to back: 2 498 -> 2 496,
// 1 263 -> 1 250, 1 048 -> 1 026, 1 370 -> 1 360, 977 -> 926.
enum class Form { Shared, Alone, Bursts };
template <int W, class R, bool UPDATE, bool WIDE, Form FORM = Form::Shared>
__global__ __launch_bounds__(kBlock, FORM == Form::Shared ? 2 : 1) void aff_mfma_kernel(float* __restrict__ params, float* __restrict__ momentum,
                                                          const RowPtrs rows, const AffCoef cf, const int64_t P,
                                                          const int head, const int span_g, const int span_k,
                                                          void* __restrict__ publish, const int publish_bf16,
                                                          double* __restrict__ partials,
                                                          const TileSource queue, const int claim,
                                                          const uint32_t period) {
    constexpr bool BURST = FORM == Form::Bursts, kAlone = FORM != Form::Shared;
    typedef GramTile<WIDE> GT;
    typedef typename GT::acc_t acc_t;
    typedef typename R::vec vec_t;
    constexpr bool BF = std::is_same<R, RowBf16x4>::value;
    constexpr int N = GT::N;
    static_assert(W <= N, "more rows than the matrix tile holds");
    constexpr int NG = W * (W + 1) / 2;
    constexpr int kWaves = kBlock / 64;
    // 17 to 24 fp32 rows: the matrix is formed group by group, four rows with four rows, for the K (K + 1) / 2 distinct
    // pairs of the K = W / 4 groups, by the instruction that multiplies 16 independent 4x4 blocks (here: 16 elements).
    // That is 480 flops per element for 20 rows and 672 for 24, where the three 16x16 blocks below take 1536 for any
    // count, at three quarters of their rate (measured: 11 to 13 cycles for 512 flops against 34 for 2048).  25.6 M
    // elements, 20 / 24 rows: norms alone 317 / 393 us, 419 / 458 by blocks, update with norms 448 / 536 against 512 / 579.
    // 28 and 32 rows need 28 and 36 pairs, whose accumulators allow one wave per SIMD only: 686 / 825 us against
    // 651 / 722 by blocks.  (One wave per SIMD with a tile of look-ahead was tried for 24 rows as well: 573.)
    // Four accumulator registers a pair leave no room for sums in double beside them; those are kept in LDS, one
    // per lane and two pairs for each wave (see fold), so that every sum is formed in a fixed order.
    constexpr bool kQuads = quad_groups(BF, W);
    constexpr int kRowStride = kQuads ? kQuadRowBytes : kPanelRowBytes;
    constexpr int kGroups = W / 4, kPairs = kQuads ? kGroups * (kGroups + 1) / 2 : 1;
    constexpr int kPanelBytes = (kQuads ? W : N) * kRowStride;
    static_assert(kPanelBytes >= 64 * 16 * 8, "the panel doubles as the reduction buffer");
    __shared__ __align__(16) unsigned char panel[kWaves][kPanelBytes];
    constexpr int kSums = (kPairs + 1) / 2 * 64;   // of a wave
    __shared__ double sums[kQuads ? kWaves * kSums : 1];
    static_assert(!kAlone || UPDATE, "a form of the update");
    constexpr int CAP = BURST ? burst_tiles_beside_panel(BF, W) : 0;
    static_assert(!BURST || sizeof(panel) + sizeof(sums) + sizeof(BurstRoom<CAP>) + 64 <= kLdsBytes, "the room fits");
    __shared__ BurstRoom<CAP> room;
    Burst<CAP> burst(room, period);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned char* const T = panel[wave];
    if constexpr (kQuads) {
        for (int i = lane; i < kSums; i += 64) sums[wave * kSums + i] = 0.0;
    } else {   // rows W..N-1 of the panel are zero and never written again
        for (int w = W; w < N; ++w) *reinterpret_cast<u32x2*>(T + w * kRowStride + 8 * lane) = u32x2{0u, 0u};
    }

    // two accumulator sets used alternately, so that consecutive matrix instructions do not wait for
    // each other's result; acc2 is the second-level sum, in double (see fold)
    acc_t acc, accb;
    double acc2[GT::REGS];
#pragma unroll
    for (int r = 0; r < GT::REGS; ++r) {
        acc[r] = 0.0f;
        accb[r] = 0.0f;
        acc2[r] = 0.0;
    }
    const unsigned char* const my_row = T + (lane % N) * kPanelRowBytes + 16 * (lane / N);
    f32x4 quad[kPairs];   // D[r][j] of pair (a, b), block n: register r of lane 4 n + j = row 4 a + r with row 4 b + j
    static_for<0, kPairs>([&](auto ec) { quad[decltype(ec)::value] = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; });
    const unsigned char* const my_quad = T + (lane % 4) * kRowStride + 16 * (lane / 4);

    // 25-32 fp32 rows: the 32x32 matrix is formed from its three distinct 16x16 blocks (rows 0-15 with
    // themselves, rows 0-15 with rows 16-31, rows 16-31 with themselves) by the 16x16x4 instruction with
    // A and B from the two halves -- three quarters of the matrix work of the 32x32x2 instruction, which
    // computes the mirrored block too and is what bounds this variant.  blk[0..2] / blkb[0..2] are the
    // alternating accumulator sets of the three blocks, blk2 their sums in double.
    constexpr bool kBlocks = WIDE && !BF && !kQuads;
    f32x4 blk[3], blkb[3];
    double blk2[12];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        blk[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        blkb[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int r = 0; r < 12; ++r) blk2[r] = 0.0;
    const unsigned char* const my_lo = T + (lane % 16) * kPanelRowBytes + 16 * (lane / 16);
    const unsigned char* const my_hi = my_lo + 16 * kPanelRowBytes;

    // stage: 512 bytes per row (8 per lane) into the panel; consume: feed them to the matrix cores.
    auto stage = [&](const u32x2 (&x)[W]) {
#pragma unroll
        for (int w = 0; w < W; ++w) *reinterpret_cast<u32x2*>(T + w * kRowStride + 8 * lane) = x[w];
    };
    auto nothing = [](auto) {};
    constexpr int kSteps = kQuads ? 8 : 512 / (16 * (kBlocks ? 4 : GT::SLOTS));   // of consume
    // `beside(step)` is vector work that the matrix instructions of a step need not wait for
    auto consume = [&](auto&& beside) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the panel is written before any lane reads it
        if constexpr (kQuads) {
            static_for<0, 512 / 256>([&](auto mc) {   // 64 elements of every row: 4 per lane, 16 lanes to a row
                constexpr int m = decltype(mc)::value;
                f32x4 y[kGroups];
#pragma unroll
                for (int a = 0; a < kGroups; ++a)
                    y[a] = *reinterpret_cast<const f32x4*>(my_quad + 4 * a * kRowStride + 256 * m);
                static_for<0, 4>([&](auto jc) {
                    constexpr int J = decltype(jc)::value;
                    static_for<0, kGroups>([&](auto ac) {
                        constexpr int A = decltype(ac)::value;
                        static_for<A, kGroups>([&](auto bc) {
                            constexpr int B = decltype(bc)::value;
                            constexpr int e = A * kGroups - A * (A - 1) / 2 + (B - A);
                            quad[e] = __builtin_amdgcn_mfma_f32_4x4x1f32(y[A][J], y[B][J], quad[e], 0, 0, 0);
                        });
                    });
                    beside(std::integral_constant<int, 4 * m + J>{});
                });
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            return;
        }
        if constexpr (kBlocks) {
#pragma unroll
            for (int m = 0; m < 512 / 64; ++m) {   // 4 slots of 16 bytes per row and step
                const f32x4 lo = *reinterpret_cast<const f32x4*>(my_lo + 64 * m);
                const f32x4 hi = *reinterpret_cast<const f32x4*>(my_hi + 64 * m);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4(&dst)[3] = (j & 1) ? blkb : blk;
                    dst[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(lo[j], lo[j], dst[0], 0, 0, 0);
                    dst[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(lo[j], hi[j], dst[1], 0, 0, 0);
                    dst[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(hi[j], hi[j], dst[2], 0, 0, 0);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            return;
        }
        typedef typename std::conditional<BF, bf16x8, f32x4>::type frag_t;
        frag_t y = *reinterpret_cast<const frag_t*>(my_row);
        static_for<0, kSteps>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            frag_t yn = y;
            if constexpr (m + 1 < kSteps) yn = *reinterpret_cast<const frag_t*>(my_row + 16 * GT::SLOTS * (m + 1));
            if constexpr (BF) {
                if (m & 1) accb = GT::mma(y, accb);
                else acc = GT::mma(y, acc);
            } else {
                acc = GT::mma(y[0], acc);
                accb = GT::mma(y[1], accb);
                acc = GT::mma(y[2], acc);
                accb = GT::mma(y[3], accb);
            }
            beside(mc);
            y = yn;
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // all reads returned before the panel is overwritten
    };
    auto gram_512 = [&](const u32x2 (&x)[W], auto&& beside) {
        // (kept apart from the update and from each other: mixed, the 24-row update spills vector registers, 578 against 542 us;
        // kept apart it spills none, the norms alone six)
        if constexpr (kQuads) __builtin_amdgcn_sched_barrier(0);
        stage(x);
        consume(beside);
        if constexpr (kQuads) __builtin_amdgcn_sched_barrier(0);
    };
    // The Gram contribution of one tile: 4 elements per lane and row.
    constexpr int kTileSteps = BF ? kSteps : 2 * kSteps;
    auto gram_tile = [&](const vec_t (&g)[W], auto&& beside) {
        if constexpr (BF) {
            gram_512(g, beside);
        } else {
            u32x2 h[W];
#pragma unroll
            for (int w = 0; w < W; ++w) h[w] = u32x2{__float_as_uint(g[w][0]), __float_as_uint(g[w][1])};
            gram_512(h, beside);
#pragma unroll
            for (int w = 0; w < W; ++w) h[w] = u32x2{__float_as_uint(g[w][2]), __float_as_uint(g[w][3])};
            gram_512(h, [&](auto mc) { beside(std::integral_constant<int, kSteps + decltype(mc)::value>{}); });
        }
    };
    // After every tile the matrix-core accumulators (256 products each by then) are folded into a
    // second set kept in double.  Two reasons.  Long fp32 chains of products of short-mantissa (bf16)
    // values drift low, about 1e-9 per term, and a tile is the natural place to cut them.  And which
    // tiles a workgroup gets from the queue differs from run to run: a tile's own sums are formed in
    // a fixed order, and adding those in double makes the order of the tiles matter only at 1e-16,
    // far below the fp32 the norms are returned in, so that they come out the same every run.
    // The fold is 4 or 16 additions per lane.
    auto fold = [&]() {
        if constexpr (kQuads) {
            // the 16 blocks of a pair's 4 registers are added four at a time by swapping halves and quarters of the wave
            // between registers: row rho of 16 lanes ends with register (0, 2, 1, 3)[rho], 4 blocks of it left.  Two pairs then
            // share a register, 2 blocks of each left: lanes 0-7 of a row the even pair, 8-15 the odd one.  Every lane adds to a
            // sum of its own.  (One addition in LDS per register and pair instead: 2-3 % slower.)
            const bool upper = (lane & 8) != 0;
            auto gathered = [&](auto ec) {
                f32x4& d = quad[decltype(ec)::value];
                const float z = swap_add<16>(swap_add<32>(d[0], d[1]), swap_add<32>(d[2], d[3]));
                d = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                return z;
            };
            static_for<0, (kPairs + 1) / 2>([&](auto hc) {
                constexpr int e = 2 * decltype(hc)::value;
                const float even = gathered(std::integral_constant<int, e>{});
                float odd = 0.0f;
                if constexpr (e + 1 < kPairs) odd = gathered(std::integral_constant<int, e + 1>{});
                const float q = (upper ? odd : even) + dpp_take<0x128, 0xf>(upper ? even : odd);   // row_ror:8
                __hip_atomic_fetch_add(&sums[wave * kSums + e * 32 + lane], (double)q, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            });
            return;
        }
        if constexpr (kBlocks) {
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    blk2[4 * b + r] += (double)(blk[b][r] + blkb[b][r]);
                    blk[b][r] = 0.0f;
                    blkb[b][r] = 0.0f;
                }
            return;
        }
#pragma unroll
        for (int r = 0; r < GT::REGS; ++r) {
            acc2[r] += (double)(acc[r] + accb[r]);
            acc[r] = 0.0f;
            accb[r] = 0.0f;
        }
    };

    // Tiles come from the queue and are walked with wave-uniform control flow (the matrix instructions
    // need every lane); a lane beyond the end of the shard contributes zeros.
    const int64_t first_tile = (int64_t)(blockIdx.x / span_g) * span_g * (int64_t)span_k + (blockIdx.x % span_g);
    const int64_t nchunk = P / 4;
    const int64_t ntile = (nchunk + kBlock - 1) / kBlock;
    // element-wise update of chunk c from values already in registers
    auto write = [&](const int64_t tile, const f32x4 (&x)[2]) {   // of a burst
        const int64_t c = tile * kBlock + threadIdx.x;
        if (c < nchunk) {
            store_through(x[0], params + tile * (4 * kBlock), threadIdx.x * 16);
            store_through(x[1], momentum + tile * (4 * kBlock), threadIdx.x * 16);
            if (publish) publish_through(x[0], publish, publish_bf16, tile);
        }
    };
    auto keep = [&](const int64_t t, const f32x4 po, const f32x4 vo) {
        const int64_t c = t * kBlock + threadIdx.x;
        if constexpr (BURST) {
            burst.put(t, {po, vo}, write);
        } else if (!kAlone || c < nchunk) {   // (Shared: only lanes of the shard get here)
            store_state(po, params, c);
            store_state(vo, momentum, c);
            if (publish) publish_chunk(po, publish, publish_bf16, c);
        }
    };
    auto update_chunk = [&](int64_t t, const vec_t (&g)[W], f32x4 pq, f32x4 vq, const AffCoef& coef) {
        if (!kAlone && t * kBlock + threadIdx.x >= nchunk) return;
        f32x4 po, vo;
        static_for<0, 4>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            float ge[W];
            static_for<0, W>([&](auto wc) {
                constexpr int Wi = decltype(wc)::value;
                ge[Wi] = R::template get<K>(g[Wi]);
            });
            float pe = pq[K], ve = vq[K];
            aff_step<W>(pe, ve, ge, coef);
            po[K] = pe;
            vo[K] = ve;
        });
        keep(t, po, vo);
    };
    auto fetch = [&](int64_t c, vec_t (&g)[W], f32x4& pq, f32x4& vq) {
        if (c < nchunk) {
#pragma unroll
            for (int w = 0; w < W; ++w) g[w] = R::load(rows.p[w], c);
            if constexpr (UPDATE) {
                pq = load_state(params, c);
                vq = load_state(momentum, c);
            }
        } else {
#pragma unroll
            for (int w = 0; w < W; ++w) g[w] = vec_t{};
        }
    };
    // The loads of the following tile are issued before this tile's update and Gram work where the Gram
    // phase is long enough to matter (not with 16 bf16 rows: 128 cycles a tile, and looking ahead measured
    // 2 % slower there) and the rows of two tiles fit in registers (up to 256 bytes per thread and tile).
    constexpr bool kAhead = sizeof(vec_t) * W <= 256 && (!BF || WIDE);   // (Shared)
    // 25 to 32 fp32 rows have no room for that, but once the second half of a tile is in the panel its registers are free, and the
    // following tile's loads go out before the matrix instructions that are left (48 updates, start -> now: 28 rows, update with norms
    // of 3 / 25.6 M elements 102 -> 95 / 646 -> 612 us, norms alone 486 -> 479; 32 rows 113 -> 107 / 719 -> 701, 545 -> 539).
    // Not with fewer: 24 rows spill 47 registers then (532 -> 595; 7 without a test around the loads, the last chunk being loaded in place
    // of those beyond the end: 530 -> 540, 3 M 84 -> 92), 20 rows lose 1 % on 80 M and their norms alone 2 % for 4 % on 3 M.
    // (Tiles worked on as two halves of 2 elements per lane and row, all of the following half's loads ahead of the matrix
    // instructions but 8 bytes each: 24 / 32 rows 531 -> 539 / 713 -> 716, norms alone 2-8 % behind.)
    constexpr bool kEarly = !kAhead && !BF && W > 24;
    if constexpr (kAlone) {
        struct Loaded {
            vec_t g[W];
            f32x4 p, v;
        } set0, set1;
        // (a lane beyond the end loads the last chunk again; its rows are cleared before they count, its results not written)
        auto load = [&](const int64_t t, Loaded& x) {
            const int64_t c = min(t * kBlock + (int64_t)threadIdx.x, nchunk - 1);
#pragma unroll
            for (int w = 0; w < W; ++w) x.g[w] = R::load(rows.p[w], c);
            x.p = load_state(params, c);
            x.v = load_state(momentum, c);
        };
        AffCoef in_vgpr = cf;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            asm volatile("" : "+v"(in_vgpr.b0[w]));
            asm volatile("" : "+v"(in_vgpr.b1[w]));
        }
        // Row groups of four have no room for the update among their matrix instructions (20 rows: 960 against 941 us).
        constexpr bool kMixed = !kQuads;
        bool primed = false;
        for_each_claimed_tile_ahead<2>(queue, ntile, claim, [&](auto sc, const int64_t t, const int64_t following) {
            constexpr int SET = decltype(sc)::value;
            Loaded& now = SET == 0 ? set0 : set1;
            Loaded& next = SET == 0 ? set1 : set0;
            const int64_t c = t * kBlock + threadIdx.x;
            if (SET == 0 && !primed) {
                load(t, now);
                primed = true;
            }
            // This tile's loads are waited for before the following one's go out.  Left to the compiler, which cannot tell on this side of
            // the branch whether those are under way, every second tile would wait for them too (16 bf16 rows, 340 M elements 2 678 us).
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            if (following >= 0) load(following, next);
            vec_t(&g)[W] = now.g;
            if (t == ntile - 1 && c >= nchunk) {
#pragma unroll
                for (int w = 0; w < W; ++w) g[w] = vec_t{};
            }
            if constexpr (kMixed) {
                // aff_step, its 4 W steps shared out over those of the matrix work
                f32x4 p = now.p, v = now.v, inc, nv;
                gram_tile(g, [&](auto mc) {
                    constexpr int S = decltype(mc)::value;
                    static_for<S * 4 * W / kTileSteps, (S + 1) * 4 * W / kTileSteps>([&](auto ic) {
                        constexpr int K = decltype(ic)::value / W, Wi = decltype(ic)::value % W;
                        if constexpr (Wi == 0) {
                            inc[K] = __builtin_fmaf(cf.m01, v[K], cf.dp * p[K]);
                            nv[K] = __builtin_fmaf(cf.m11, v[K], cf.m10 * p[K]);
                        }
                        const float x = R::template get<K>(g[Wi]);
                        inc[K] = __builtin_fmaf(in_vgpr.b0[Wi], x, inc[K]);
                        nv[K] = __builtin_fmaf(in_vgpr.b1[Wi], x, nv[K]);
                        if constexpr (Wi == W - 1) p[K] = p[K] + inc[K];
                    });
                    if constexpr (!BF) __builtin_amdgcn_sched_barrier(0);   // (bf16 rows, 8 or 16 matrix instructions a tile: better without)
                });
                fold();
                keep(t, p, nv);
            } else {
                update_chunk(t, g, now.p, now.v, in_vgpr);
                gram_tile(g, nothing);
                fold();
            }
        });
    } else if constexpr (kAhead) {
        vec_t gn[W];
        f32x4 pn = {0, 0, 0, 0}, vn = {0, 0, 0, 0};
        bool primed = false;
        for_each_claimed_tile_ahead(queue, ntile, claim, [&](const int64_t t, const int64_t following) {
            const int64_t c = t * kBlock + threadIdx.x;
            if (!primed) {
                fetch(c, gn, pn, vn);
                primed = true;
            }
            vec_t g[W];
#pragma unroll
            for (int w = 0; w < W; ++w) g[w] = gn[w];
            const f32x4 pq = pn, vq = vn;
            if (following >= 0) fetch(following * kBlock + threadIdx.x, gn, pn, vn);
            if constexpr (UPDATE) update_chunk(t, g, pq, vq, cf);
            gram_tile(g, nothing);
            fold();
        });
    } else if constexpr (kEarly) {
        vec_t g[W];
        f32x4 pq = {0, 0, 0, 0}, vq = {0, 0, 0, 0};
        bool primed = false;
        for_each_claimed_tile_ahead(queue, ntile, claim, [&](const int64_t t, const int64_t following) {
            const int64_t c = t * kBlock + threadIdx.x;
            if (!primed) {
                fetch(c, g, pq, vq);
                primed = true;
            }
            if constexpr (UPDATE) update_chunk(t, g, pq, vq, cf);
            u32x2 h[W];   // gram_tile, with the loads before its last step
#pragma unroll
            for (int w = 0; w < W; ++w) h[w] = u32x2{__float_as_uint(g[w][0]), __float_as_uint(g[w][1])};
            gram_512(h, nothing);
#pragma unroll
            for (int w = 0; w < W; ++w) h[w] = u32x2{__float_as_uint(g[w][2]), __float_as_uint(g[w][3])};
            stage(h);
            if (following >= 0) fetch(following * kBlock + threadIdx.x, g, pq, vq);
            consume(nothing);
            fold();
        });
    } else {
        for_each_claimed_tile(queue, ntile, claim, [&](const int64_t t) {
            const int64_t c = t * kBlock + threadIdx.x;
            vec_t g[W];
            f32x4 pq = {0, 0, 0, 0}, vq = {0, 0, 0, 0};
            fetch(c, g, pq, vq);
            if constexpr (UPDATE) update_chunk(t, g, pq, vq, cf);
            gram_tile(g, nothing);
            fold();
        });
    }
    if constexpr (BURST) burst.flush(write);
    // elements not covered by whole chunks: one element per lane, same arithmetic
    const int64_t nrest = rest_count(head, P, nchunk);
    const int64_t nrtile = (nrest + kBlock - 1) / kBlock;
    int64_t tile = first_tile;
    for (int k = 0; k < span_k && tile < nrtile; ++k, tile += span_g) {
        const int64_t r = tile * kBlock + threadIdx.x;
        vec_t g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) g[w] = vec_t{};
        if (r < nrest) {
            const int64_t j = rest_element(r, head, nchunk);
            float g1[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                g1[w] = R::load1(rows.p[w], j);
                if constexpr (BF) g[w][0] = __float_as_uint(g1[w]) >> 16;   // exact: the value came from a bf16
                else g[w][0] = g1[w];
            }
            if constexpr (UPDATE) {
                float pj = params[j], vj = momentum[j];
                aff_step<W>(pj, vj, g1, cf);
                params[j] = pj;
                momentum[j] = vj;
                if (publish) publish_element(pj, publish, publish_bf16, j);
            }
        }
        gram_tile(g, nothing);
        fold();
    }

    // workgroup total of every Gamma entry, in double, one partial per workgroup; each wave's
    // accumulators go through its own (now idle) panel (kQuads: they are in `sums` already)
    double* const red = reinterpret_cast<double*>(T);
    if constexpr (kBlocks) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[lane * 12 + 4 * b + r] = (double)(blk[b][r] + blkb[b][r]) + blk2[4 * b + r];
    } else if constexpr (!kQuads) {
#pragma unroll
        for (int r = 0; r < GT::REGS; ++r) red[lane * GT::REGS + r] = (double)(acc[r] + accb[r]) + acc2[r];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NG; e += kBlock) {
        int i = 0, rem = e;
        while (rem >= W - i) {
            rem -= W - i;
            ++i;
        }
        const int j = i + rem;
        double s = 0.0;
        if constexpr (kQuads) {
            const int a = i / 4, b = j / 4;
            const int r = i % 4, rho = 2 * (r & 1) + r / 2;
            const int e2 = a * kGroups - a * (a - 1) / 2 + (b - a);   // the pair
            const double* src = sums + (e2 / 2) * 64 + 16 * rho + 8 * (e2 % 2) + j % 4;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) s += src[q * kSums] + src[q * kSums + 4];
        } else {
            int src;
            if constexpr (kBlocks) {
                // entry (i, j), i <= j, lies in block 0 (both below 16), 1 (i below, j from 16 on) or 2; inside a
                // block, D[a][b] is register a % 4 of lane 16 * (a / 4) + b
                const int b = (i >= 16) ? 2 : (j >= 16 ? 1 : 0);
                const int a = i & 15, c = j & 15;
                src = (16 * (a / 4) + c) * 12 + 4 * b + (a % 4);
            } else {
                src = GT::lane_of(i, j) * GT::REGS + GT::reg_of(i);
            }
#pragma unroll
            for (int q = 0; q < kWaves; ++q) s += reinterpret_cast<const double*>(panel[q])[src];
        }
        partials[(int64_t)e * gridDim.x + blockIdx.x] = s;
    }
}

namespace {

template <int W, class R, bool UPDATE, bool WIDE>
hipError_t launch_mfma_t(const AffArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    auto kern = aff_mfma_kernel<W, R, UPDATE, WIDE>;
    // Long-lived workgroups, tiles from the queue.  Two per compute unit, so that one wave's Gram phase overlaps
    // another's loads; one where a single workgroup already keeps about 48 KB and more in flight, looks a
    // tile ahead and writes the state (10 to 16 fp32 rows: 2-5 % faster with one, e.g. 16 rows 1.51 against
    // 1.56 ms on the 110 M shard; 8 rows no difference; the norms alone, a pure read, run 1.13 against
    // 1.24 ms with two).  The LDS panels (33 KB narrow, 66 KB
    // wide per workgroup) allow both.
    // 20 to 32 bf16 rows, update: one as well from the length on at which the two would take claims (8 / 30 / 120 M elements,
    // 20 rows: 94 / 299 / 1133 against 101 / 308 / 1164 us, 32 rows: 136 / 448 / 1705 against 145 / 461 / 1757; but 3 M,
    // 32 rows: 69 against 65, and 17 rows, whose padding costs no traffic, 30 M: 284 against 278).
    constexpr int kRowBytes = W * (int)sizeof(typename R::vec);
    constexpr bool kBf16 = std::is_same<R, RowBf16x4>::value;
    const int64_t tiles = tiles_of(a.P);
    const bool one_wide = UPDATE && WIDE && kBf16 && a.rows_used >= 20 &&
                          tiles > 2 * (int64_t)num_cu * short_tiles_per_workgroup(kRowBytes + 32, Traffic::Update);
    // 8 and 9 fp32 rows, update, from 16 Mi elements on: one too (18 / 60 M elements, 8 rows 161.7 / 487 -> 152.9 / 470 us, 60 M, 9 rows 539 -> 507).  After
    // a pause the first call is level (8 / 9 rows 548 / 597 -> 551 / 594 us), those of 3 to 15 ms later lose 4-8 %, see Form.  Not 7 rows: 448 against
    // 457, the first call after a pause 549 against 576.
    constexpr bool kLight = UPDATE && !WIDE && !kBf16 && (W == 8 || W == 9);
    const bool one_light = kLight && tiles >= 16 * 1024;
    const int per_cu = (UPDATE && !WIDE && kRowBytes >= 160) || one_wide || one_light ? 1 : 2;
    if (!a.queue) return hipErrorInvalidValue;
    Geometry g = queue_geometry(num_cu, grid_cap, per_cu, kRowBytes + (UPDATE ? 32 : 0),
                                UPDATE ? Traffic::Update : Traffic::ReadOnly, tiles);
    // The norms of 17 to 32 bf16 rows: one workgroup per unit, whose look-ahead keeps 64 KB in flight, and the tiles split
    // evenly up to 256 a workgroup (3 / 30 / 60 M elements, 24 rows: 36.8 / 224 / 426 against 38.8 / 232 / 438 us, 32 rows:
    // 46 / 294 / 566 against 48 / 302 / 575; 120 M, 32 rows: 1127 against 1119), up to 20 rows up to 128 (20 rows, 26 / 40 M 162 /
    // 258 against 169 / 249; 17 rows, 60 M 335 against 325).
    if (!UPDATE && WIDE && kBf16 && tiles <= (W <= 20 ? 128 : 256) * (int64_t)num_cu) {
        g.claim = -1;
        g.grid = g.span_g = (int)std::max<int64_t>(1, std::min<int64_t>(std::min(num_cu, grid_cap), tiles));
    }
    if constexpr (UPDATE && mfma_bursts(W, !kBf16)) {
        if (a.burst) {
            const int grid = (int)std::min<int64_t>(std::min(num_cu, grid_cap), std::max<int64_t>(1, tiles));
            *grid_out = grid;
            hipLaunchKernelGGL((aff_mfma_kernel<W, R, UPDATE, WIDE, Form::Bursts>), dim3(grid), dim3(kBlock), 0, s, a.params, a.momentum, a.rows,
                               a.cf, a.P, a.head, grid, 0x7fffffff, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0, a.partials,
                               TileSource{a.queue, nullptr, 0u}, a.burst,
                               burst_period(burst_tiles_beside_panel(kBf16, W), (kRowBytes + 64 + copy_bytes(a)) * kBlock, grid, 0.9));
            return hipGetLastError();
        }
    }
    *grid_out = g.grid;
    if constexpr (kLight) {
        if (one_light) kern = aff_mfma_kernel<W, R, UPDATE, WIDE, Form::Alone>;
    }
    hipLaunchKernelGGL(kern, dim3(g.grid), dim3(kBlock), 0, s, a.params, a.momentum, a.rows, a.cf, a.P, a.head,
                       g.span_g, g.span_k, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0, a.partials,
                       TileSource{a.queue, nullptr, 0u}, g.claim, 0u);
    return hipGetLastError();
}

template <int W>
hipError_t launch_mfma_w(int dtype, bool update, const AffArgs& a, int num_cu, int grid_cap, int* grid_out,
                         hipStream_t s) {
    constexpr bool WIDE = W > 16;
    if (dtype == STAR_F32) {
        if (update) return launch_mfma_t<W, RowF32, true, WIDE>(a, num_cu, grid_cap, grid_out, s);
        return launch_mfma_t<W, RowF32, false, WIDE>(a, num_cu, grid_cap, grid_out, s);
    }
    if (update) return launch_mfma_t<W, RowBf16x4, true, WIDE>(a, num_cu, grid_cap, grid_out, s);
    return launch_mfma_t<W, RowBf16x4, false, WIDE>(a, num_cu, grid_cap, grid_out, s);
}

}  // namespace

hipError_t launch_affine_mfma(int Wp, int dtype, bool update, const AffArgs& a, int num_cu, int grid_cap,
                              int* grid_out, hipStream_t s) {
    switch (Wp) {
#define X(N) case N: return launch_mfma_w<N>(dtype, update, a, num_cu, grid_cap, grid_out, s);
        STAR_FOR_EACH_W(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace star
