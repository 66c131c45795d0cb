// gfx950 kernel: direct sums of gbar_u^2 on the matrix cores, see norm_mma_kernel.  A header, because the two row types are
// compiled as two files: 32 kernels each, about a minute.
#pragma once

#include "star_device.h"

namespace star {

// Constant address space: uniform reads become scalar loads.  The tables are written before the launch and not during it.
#define STAR_CONST __attribute__((address_space(4)))

struct WalkKernelArgs {
    RowPtrs rows;
    const float* coef;      // [U][W], or null: the tables are in `inl`
    const uint32_t* mask;   // [U]
    double* partials;
    int64_t P;
    int32_t U, head;
    int32_t share;          // updates per workgroup, see launch_walk_t
    InlineTables inl;
};

hipError_t launch_norm_mma_f32(WalkKernelArgs& k, int Wp, int num_cu, int grid_cap, int* grid_out, hipStream_t s);
hipError_t launch_norm_mma_bf16(WalkKernelArgs& k, int Wp, int num_cu, int grid_cap, int* grid_out, hipStream_t s);

// gbar is a product, [updates x rows] times [rows x elements], and the fp32 matrix instructions multiply at twice the rate
// the vector ALUs reach without packed instructions; what is left for those are the squares.
//   v_mfma_f32_16x16x4_f32 takes 16 updates x 4 rows from A and 4 rows x 16 elements from B.  Lane l feeds row 4 s + l / 16
// and the element l % 16 of its 16, so that a lane's 16-byte load, 4 or 8 elements of one row, is the B operand of 4 or 8
// instructions as it stands: no transposition, no LDS.  Lane l of the result holds updates 4 (l / 16) + r, r = 0 .. 3, of
// one element, so every lane squares and sums on its own, and the lanes meet once, when the kernel ends.
//   The multiplication is dense: a row that is no member of a group enters with coefficient zero.  That is the same sum, except
// where the row holds an infinity or a NaN; tiles that do are found beforehand (x * 0 is not 0), see Odd.
//   bf16 rows: v_mfma_f32_16x16x32_bf16, at 16 times the rate.  The coefficients stay fp32 numbers, as the sum of three bf16 pieces
// each (products of two bf16 values are exact in fp32, where they are added).  A lane's eight places of the reduction are four
// pairs of rows, once for every piece, packed from the loads of two row groups by one instruction an element.
//   The upper pieces have an instruction to themselves.  The instruction adds the eight products of a quarter of the wave at a time
// and cuts off, instead of rounding, what lies more than 25 bits below the largest: all three pieces in one made the norms of up to 8 rows 1.5e-8
// too small on the mean.  The lower two come first, so that the large products are rounded once: gbar of normal rows is then off by
// 3.5e-8 of its size whatever the row count (fp32 multiply-adds, norm_walk_kernel: 2.5e-8 / 4e-8 / 6e-8 / 9e-8 with 1 / 6 / 16 / 32
// rows).  Up to four rows the upper ones come first, 2.5e-8 with one row.  What the norm of 65 536 normal elements is off by for that, before it is rounded
// to fp32: 0.3e-9 to 3e-9 rms (multiply-adds: 0.7e-9 to 2e-9); rows of one sign up to 1.5e-8 (6e-9).
//   It costs up to 8 rows an instruction more (30 M elements, 4 / 8 rows, 32 updates 82 / 96 -> 102 / 118 us, norm_walk_kernel 134 / 220).
//   Memory bounds it, within 8 %, with 16 updates from 8 fp32 or 16 bf16 rows on and with 32 updates of 32 bf16 rows; beyond, the matrix
// instructions and the squares do, which overlap only in part.  25.6 M elements, norm_walk_kernel -> this one (the reads alone): 8 fp32 rows, 32 updates of
// 4.5 members 198 -> 160 us (120), 16 rows, 16 / 32 updates 302 / 424 -> 251 / 274 (240), 32 rows, 16 updates 717 -> 498 (481); bf16 rows: 8 rows, 32
// updates 206 -> 105 (60), 16 rows, 16 / 64 updates 239 / 722 -> 128 / 208 (120), 30 M, 32 rows, 32 updates 1437 -> 311 (282).  bf16 rows through the fp32
// instructions, 30 M: 8 rows, 32 updates 167, 16 rows, 64 updates 540, 32 rows, 64 updates 1042.
//   Largest error of a norm against 64 bits, 1 to 32 rows, 3 to 240 updates: 9.7e-8 either way for fp32 rows, bf16 rows 6.3e-8 either way.
typedef float acc4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));

// 16 bytes of a row: one load of a lane
template <class R>
struct WideLoad;
template <>
struct WideLoad<RowF32> {
    static constexpr int E = 4;
    typedef f32x4 vec;
    static __device__ __forceinline__ vec load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
    }
};
template <>
struct WideLoad<RowBf16x4> {
    static constexpr int E = 8;
    typedef u32x4 vec;
    static __device__ __forceinline__ vec load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
    }
};

// The three bf16 values that add up to an fp32 coefficient: its upper eight bits, the next eight, the rest.
__device__ __forceinline__ uint32_t coef_piece(float c, const int piece) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (i < piece) c -= __uint_as_float(__float_as_uint(c) & 0xffff0000u);   // exact
    return __float_as_uint(c) >> 16;
}

// 16-byte loads per lane and row group of a tile: about 8 KB of a wave in flight, and as much again from the look-ahead.
constexpr int mma_units(int KS) { return KS == 1 ? 8 : (KS == 2 ? 4 : (KS <= 4 ? 2 : 1)); }

// Waves per SIMD the registers are cut for, and the launch made for: three with one block of updates, and with two up to 16 rows.  (Most of the other
// fp32 instances would have registers for three as well, 117 to 167; only 8 rows, 32 updates were timed both ways, see launch_mma_k.)
constexpr int mma_waves(int KS, int NB) { return NB == 1 || (NB == 2 && KS <= 4) ? 3 : 2; }

// KS row groups of four, NB blocks of 16 updates
template <int KS, int NB, class R>
__global__ __launch_bounds__(kBlock, mma_waves(KS, NB)) void norm_mma_kernel(const WalkKernelArgs args, const int W) {
    typedef WideLoad<R> L;
    typedef typename L::vec vec_t;
    constexpr int E = L::E, CH = mma_units(KS);
    constexpr int kUnit = 16 * E;            // elements of a unit: 16 lanes, one load each
    constexpr int kTile = kUnit * CH;        // elements of a wave's tile
    constexpr int kRowWaves = kBlock / 64;
    const int u0 = (int)blockIdx.y * args.share, U = min(args.U - u0, args.share);
    const auto* const in = (const STAR_CONST WalkKernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const STAR_CONST float* coef = (const STAR_CONST float*)args.coef;
    const STAR_CONST uint32_t* mask = (const STAR_CONST uint32_t*)args.mask;
    if (!args.coef) {
        coef = in->inl.coef;
        mask = in->inl.mask;
    }
    coef += u0 * W;
    mask += u0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quarter = lane >> 4, col = lane & 15;

    // operand A: zero beyond the last update and the last row
    auto coef_at = [&](const int u, const int s) {
        const int w = 4 * s + quarter;
        return s < KS && u < U && w < W ? coef[u * W + w] : 0.0f;
    };
    constexpr bool BF = std::is_same<R, RowBf16x4>::value;
    constexpr int kPairs = (KS + 1) / 2, kLow = (2 * kPairs + 3) / 4, kSteps = BF ? kLow + 1 : KS;
    constexpr int kHigh = KS > 1 ? kLow : 0;   // the step of the upper pieces, see bf16 rows above
    typedef typename std::conditional<BF, bf16x8, float>::type operand_t;
    operand_t a[NB][kSteps];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int u = 16 * b + col;
        if constexpr (BF) {
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                u32x4 packed;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int slot = i == kHigh ? p : 4 * (i - (KS > 1 ? 0 : 1)) + p;
                    const int pair = slot % kPairs, piece = i == kHigh ? 0 : 1 + slot / kPairs;
                    const bool used = slot < (i == kHigh ? 1 : 2) * kPairs;
                    const uint32_t lo = used ? coef_piece(coef_at(u, 2 * pair), piece) : 0u;
                    const uint32_t hi = used ? coef_piece(coef_at(u, 2 * pair + 1), piece) : 0u;
                    packed[p] = hi << 16 | lo;
                }
                a[b][i] = __builtin_bit_cast(bf16x8, packed);
            }
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) a[b][s] = coef_at(u, s);
        }
    }
    const char* row[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) row[s] = reinterpret_cast<const char*>(in->rows.p[4 * s + quarter]);

    double sum[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[b][r] = 0.0;

    const int64_t P = args.P, nchunk = P / E;   // chunks: one lane's load
    const int64_t ntile = (nchunk + kTile / E - 1) / (kTile / E);
    // Infinities and NaN: a dense product would carry them into every group (0 times either is NaN).  They are taken out of the
    // operand, and what they make of their groups is kept apart, as two sets of updates that the sums meet when the kernel ends.  From which
    // rows of a tile hold NaN, +inf or -inf (`Odd`, bits of rows) most of it follows without a look at the elements, one update a
    // lane: a member with NaN, or with an infinity and a coefficient of zero, makes the sum NaN; infinities that all enter a group with
    // the same sign, or that are one row's, make it infinite.  Only where rows meet in a group with infinities of both signs and its sum is
    // not NaN yet are they looked at element by element (poison).  What a wave has seen once needs no second look: rows with NaN, since
    // the sums they are in are NaN, and infinite rows while no group has a choice of signs.  So a worker that diverged costs the wave one tile
    // and the others little more than the search (8 rows of 25.6 M elements, 32 updates, clean / one row of NaN / of +inf / of infinities of both signs / all
    // rows of +inf: fp32 166 / 229 / 208 / 205 / 192 us, bf16 105 / 153 / 148 / 146 / 137; two rows that agree in signs that change 267, 251;
    // norm_walk_kernel 197 to 220 and 187 to 207; every spoilt tile element by element: 1460 to 2870 us).
    uint64_t lost = 0, infinite = 0;   // updates whose sum is NaN; whose sum is infinite at least
    struct Odd {
        uint32_t nan, pos, neg;
    };
    Odd seen = {0, 0, 0};
    // One update a lane: takes in what a tile holds; the updates whose infinite members must be looked at element by element, and the
    // members by the signs of their coefficients.
    auto examine = [&](const Odd& o, uint32_t& plus, uint32_t& minus) {
        const uint32_t pos = o.pos | seen.pos, neg = o.neg | seen.neg;
        const uint32_t m = lane < U ? mask[lane] : 0u;
        bool nan = (m & o.nan) != 0;
        plus = minus = 0;
        for (uint32_t left = pos | neg; left; left &= left - 1) {
            const uint32_t w = __builtin_ctz(left), bit = m & (1u << w);
            const float c = bit ? coef[lane * W + w] : 1.0f;
            nan = nan || c == 0.0f;
            (c < 0.0f ? minus : plus) |= bit;
        }
        const uint32_t up = (plus & pos) | (minus & neg), down = (plus & neg) | (minus & pos);   // members that add +inf, -inf
        lost |= __builtin_amdgcn_ballot_w64(nan);
        infinite |= __builtin_amdgcn_ballot_w64((up | down) != 0);
        auto meet = [](const uint32_t a, const uint32_t b) { return a && b && ((a | b) & ((a | b) - 1)); };
        const uint64_t open = __builtin_amdgcn_ballot_w64(meet(up, down)) & ~lost;
        seen.nan |= o.nan;
        if (!open) {
            seen.pos = pos;
            seen.neg = neg;
        }
        const uint32_t here = o.pos | o.neg;
        return __builtin_amdgcn_ballot_w64(meet(up & here, down & here)) & open;
    };
    // The updates `todo` whose infinite members are of both signs at an element: `n` times 64 of them, one per lane, at(i) the i-th
    // (INT64_MIN: none).  Most rows agree in sign wherever they are infinite, which settles the groups whose coefficients do.
    auto poison = [&](auto at, auto n, const uint32_t rows, const uint64_t todo, const uint32_t plus, const uint32_t minus) {
        constexpr int N = decltype(n)::value, Q = N < 4 ? N : 4;   // Q loads in flight
        const uint64_t mixed = __builtin_amdgcn_ballot_w64((plus & rows) && (minus & rows)) & todo;
#pragma unroll 1
        for (int i = 0; i < N; i += Q) {
            uint32_t pos[Q], neg[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) pos[q] = neg[q] = 0u;
#pragma unroll 1
            for (uint32_t left = rows; left; left &= left - 1) {
                const uint32_t w = __builtin_ctz(left);
                const void* const row = in->rows.p[w];
                float v[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) v[q] = at(i + q) != INT64_MIN ? R::load1(row, at(i + q)) : 0.0f;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    pos[q] |= v[q] == __builtin_inff() ? 1u << w : 0u;
                    neg[q] |= v[q] == -__builtin_inff() ? 1u << w : 0u;
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint32_t any = pos[q] | neg[q];
                if (!__builtin_amdgcn_ballot_w64((any & (any - 1)) != 0)) continue;   // two rows nowhere
                const bool agree = !__builtin_amdgcn_ballot_w64(pos[q] && neg[q]);
                for (uint64_t left = (agree ? mixed : todo) & ~lost; left; left &= left - 1) {
                    const int u = __builtin_ctzll(left);
                    const uint32_t a = __builtin_amdgcn_readlane(plus, u), b = __builtin_amdgcn_readlane(minus, u);
                    if (__builtin_amdgcn_ballot_w64(((pos[q] & a) | (neg[q] & b)) && ((pos[q] & b) | (neg[q] & a))))
                        lost |= 1ull << u;
                }
            }
        }
    };
    // What a lane has of the rows' kinds: the largest bits of all, and as a signed number, by magnitude and as an unsigned one.  (With NaN
    // the infinities beside them may be hidden, or seen where there are none: the sums of such a row are NaN.)
    typedef typename std::conditional<BF, u16x2, uint32_t>::type bits_t;
    typedef typename std::conditional<BF, i16x2, int32_t>::type sbits_t;
    struct Kinds {
        bits_t size, last;
        sbits_t first;
    };
    auto none = [&]() {
        if constexpr (BF) return Kinds{u16x2{0, 0}, u16x2{0, 0}, i16x2{0, 0}};
        else return Kinds{0u, 0u, 0};
    };
    auto clean = [&](vec_t& x, Kinds& kd) {   // takes them out of one load
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (BF) {
                const uint32_t d = x[k];
                kd.size = __builtin_elementwise_max(kd.size, __builtin_bit_cast(u16x2, d & 0x7fff7fffu));
                kd.last = __builtin_elementwise_max(kd.last, __builtin_bit_cast(u16x2, d));
                kd.first = __builtin_elementwise_max(kd.first, __builtin_bit_cast(i16x2, d));
                const bool lo = (d & 0x7f80u) == 0x7f80u, hi = (d & 0x7f800000u) == 0x7f800000u;
                x[k] = (lo ? 0u : d & 0xffffu) | (hi ? 0u : d & 0xffff0000u);
            } else {
                const uint32_t d = __float_as_uint(x[k]);
                kd.size = max(kd.size, d & 0x7fffffffu);
                kd.last = max(kd.last, d);
                kd.first = max(kd.first, (int32_t)d);
                x[k] = (d & 0x7f800000u) == 0x7f800000u ? 0.0f : x[k];
            }
        }
    };
    auto rows_of = [&](const bool any, const int s) {   // rows 4 s .. 4 s + 3 by the quarters of the wave that held any
        const uint64_t lanes = __builtin_amdgcn_ballot_w64(any);
        uint32_t rows = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) rows |= (lanes >> (16 * q) & 0xffffu) ? 1u << (4 * s + q) : 0u;
        return W < 32 ? rows & ((1u << W) - 1u) : rows;   // (beyond the last row it is repeated)
    };
    auto add_kinds = [&](Odd& o, const Kinds& kd, const int s) {
        if constexpr (BF) {
            o.nan |= rows_of(kd.size[0] > 0x7f80 || kd.size[1] > 0x7f80, s);
            o.pos |= rows_of(kd.first[0] >= 0x7f80 || kd.first[1] >= 0x7f80, s);
            o.neg |= rows_of(kd.last[0] >= 0xff80 || kd.last[1] >= 0xff80, s);
        } else {
            o.nan |= rows_of(kd.size > 0x7f800000u, s);
            o.pos |= rows_of(kd.first >= 0x7f800000, s);
            o.neg |= rows_of(kd.last >= 0xff800000u, s);
        }
    };
    auto news = [&](const Odd& o) {   // what no earlier tile has settled
        return ((o.nan | (o.pos & ~seen.pos) | (o.neg & ~seen.neg)) & ~seen.nan) != 0;
    };

    auto fetch = [&](const int64_t tile, vec_t (&x)[CH][KS]) {
        const int64_t c0 = tile * (kTile / E) + col;
        if ((tile + 1) * (kTile / E) <= nchunk) {
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int s = 0; s < KS; ++s) x[c][s] = L::load(row[s] + (c0 + 16 * c) * 16);
        } else {   // the last tile: lanes beyond the end read the last chunk and hold zeros
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int64_t at = c0 + 16 * c, from = at < nchunk ? at : nchunk - 1;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    x[c][s] = L::load(row[s] + from * 16);
                    if (at >= nchunk) x[c][s] = vec_t{};
                }
            }
        }
    };
    // a unit: one load of every row group
    auto product = [&](const vec_t (&x)[KS]) {
        static_for<0, E / 4>([&](auto hc) {   // four elements of a lane at a time: four squares in fp32
            constexpr int H = decltype(hc)::value;
            uint32_t pk[4][kPairs];   // two rows' values of one element
            if constexpr (BF) {
                static_for<0, 4>([&](auto kc) {
                    constexpr int K = decltype(kc)::value, D = 2 * H + K / 2;
                    static_for<0, kPairs>([&](auto pc) {
                        constexpr int S = 2 * decltype(pc)::value, T = S + 1 < KS ? S + 1 : S;
                        pk[K][S / 2] = __builtin_amdgcn_perm(x[T][D], x[S][D], K & 1 ? 0x07060302u : 0x05040100u);
                    });
                });
            }
            static_for<0, NB>([&](auto bc) {
                constexpr int B = decltype(bc)::value;
                acc4 d[4];
                static_for<0, 4>([&](auto kc) { d[decltype(kc)::value] = acc4{0.0f, 0.0f, 0.0f, 0.0f}; });
                static_for<0, kSteps>([&](auto sc) {
                    constexpr int S = decltype(sc)::value;
                    static_for<0, 4>([&](auto kc) {
                        constexpr int K = decltype(kc)::value;
                        if constexpr (BF) {
                            constexpr int F = S == kHigh ? 0 : 4 * (S - (KS > 1 ? 0 : 1));   // its first place, as above
                            const u32x4 y = {pk[K][F % kPairs], pk[K][(F + 1) % kPairs], pk[K][(F + 2) % kPairs],
                                             pk[K][(F + 3) % kPairs]};
                            d[K] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[B][S], __builtin_bit_cast(bf16x8, y), d[K], 0, 0,
                                                                           0);
                        } else {
                            d[K] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[B][S], x[S][K], d[K], 0, 0, 0);
                        }
                    });
                });
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float sq = 0.0f;
#pragma unroll
                    for (int k = 0; k < 4; ++k) sq = __builtin_fmaf(d[k][r], d[k][r], sq);
                    sum[B][r] += (double)sq;
                }
            });
        });
    };
    // an infinity or a NaN among them: fp32 x * 0 is NaN then, bf16 an exponent of all ones
    float odd;
    u16x2 most;
    auto look = [&](const vec_t& x) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (BF) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, x[k] & 0x7fff7fffu));
            else odd = __builtin_fmaf(x[k], 0.0f, odd);
        }
    };
    auto spoilt = [&]() {
        const bool any = BF ? most[0] >= 0x7f80 || most[1] >= 0x7f80 : odd != odd;
        return __builtin_expect(__builtin_amdgcn_ballot_w64(any) != 0, 0);
    };
    const int64_t step = (int64_t)gridDim.x * kRowWaves;
    int64_t tile = (int64_t)blockIdx.x * kRowWaves + wave;
    vec_t next[CH][KS];
    if (tile < ntile) fetch(tile, next);
    for (; tile < ntile; tile += step) {
        vec_t x[CH][KS];
        odd = 0.0f;
        most = u16x2{0, 0};
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                x[c][s] = next[c][s];
                look(x[c][s]);
            }
        if (tile + step < ntile) fetch(tile + step, next);
        if (spoilt()) {
            Odd o = {0, 0, 0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                Kinds kd = none();
#pragma unroll
                for (int c = 0; c < CH; ++c) clean(x[c][s], kd);
                add_kinds(o, kd, s);
            }
            if (news(o)) {
                uint32_t plus, minus;
                const uint64_t todo = examine(o, plus, minus);
                if (todo) {
                    auto at = [&](const int i) {
                        const int64_t j = tile * kTile + 64 * i + lane;
                        return j < nchunk * E ? j : INT64_MIN;
                    };
                    poison(at, std::integral_constant<int, kTile / 64>{}, o.pos | o.neg, todo, plus, minus);
                }
            }
        }
        static_for<0, CH>([&](auto cc) {
            constexpr int C = decltype(cc)::value;
            product(x[C]);
            // fp32 rows: the units are scheduled in two halves (in one, the registers run out with 8 rows and 32 updates: 159 -> 180 us)
            if constexpr (!BF && 2 * C + 2 == CH) __builtin_amdgcn_sched_barrier(0);
        });
    }
    // What the chunks leave over, at most 63 + 7 elements, for the wave whose turn it is: fetched one by one, then a unit like the
    // others (walked instead, they take half a microsecond an update: 0.3 M elements, 8 rows, 64 updates 49 against 23 us).
    if (tile == ntile) {
        const int64_t nrest = args.head + (P - nchunk * E);
        auto rest = [&](const int64_t r) { return r < args.head ? r - args.head : nchunk * E + (r - args.head); };
#pragma unroll 1
        for (int64_t r0 = 0; r0 < nrest; r0 += kUnit) {
            vec_t x[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) x[s] = vec_t{};
#pragma unroll 1
            for (int e = 0; e < E; ++e) {   // element e enters from above, the others move down by one
                const int64_t r = r0 + col * E + e, j = rest(r < nrest ? r : nrest - 1);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    if constexpr (BF) {
                        const uint32_t v = r < nrest ? reinterpret_cast<const uint16_t*>(row[s])[j] : 0u;
#pragma unroll
                        for (int k = 0; k < 4; ++k) x[s][k] = x[s][k] >> 16 | (k < 3 ? x[s][k + 1] : v) << 16;
                    } else {
                        const float v = r < nrest ? reinterpret_cast<const float*>(row[s])[j] : 0.0f;
                        x[s] = vec_t{x[s][1], x[s][2], x[s][3], v};
                    }
                }
            }
            odd = 0.0f;
            most = u16x2{0, 0};
#pragma unroll
            for (int s = 0; s < KS; ++s) look(x[s]);
            if (spoilt()) {
                Odd o = {0, 0, 0};
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    Kinds kd = none();
                    clean(x[s], kd);
                    add_kinds(o, kd, s);
                }
                uint32_t plus = 0, minus = 0;
                const uint64_t todo = news(o) ? examine(o, plus, minus) : 0;
                if (todo) {
                    auto at = [&](const int i) { return r0 + 64 * i + lane < nrest ? rest(r0 + 64 * i + lane) : INT64_MIN; };
                    poison(at, std::integral_constant<int, kUnit / 64>{}, o.pos | o.neg, todo, plus, minus);
                }
            }
            product(x);
        }
    }

    // 16 lanes hold parts of the same four updates: summed within the 16, then over the waves, in a fixed order
    __shared__ double total[kRowWaves][16 * NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double q = sum[b][r];
            q += dpp_take<0xB1, 0xf>(q);    // quad_perm [1,0,3,2]
            q += dpp_take<0x4E, 0xf>(q);    // quad_perm [2,3,0,1]
            q += dpp_take<0x141, 0xf>(q);   // row_half_mirror
            q += dpp_take<0x140, 0xf>(q);   // row_mirror
            if (col == 0) total[wave][16 * b + 4 * quarter + r] = q;
        }
    if (lost | infinite) {   // one update a lane
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if ((lost >> lane) & 1u) total[wave][lane] = __builtin_nan("");   // (no bit is set beyond the last update)
        else if ((infinite >> lane) & 1u) total[wave][lane] += __builtin_inf();
    }
    __syncthreads();
    for (int u = threadIdx.x; u < U; u += kBlock) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < kRowWaves; ++q) s += total[q][u];
        args.partials[(int64_t)(u0 + u) * gridDim.x + blockIdx.x] = s;
    }
}

template <int KS, class R>
hipError_t launch_mma_k(WalkKernelArgs& k, int W, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    constexpr int kTile = 16 * WideLoad<R>::E * mma_units(KS) * (kBlock / 64);   // elements of a workgroup's tile
    const int64_t tiles = std::max<int64_t>(1, (k.P + kTile - 1) / kTile + (k.head ? 1 : 0));
    // More than 64 updates, or a shard of fewer tiles than units: the updates are shared out over workgroups, in blocks of 16.
    const int blocks = (k.U + 15) / 16;
    const int parts = std::max((blocks + 3) / 4, (int)std::min<int64_t>(blocks, std::max<int64_t>(1, num_cu / tiles)));
    const int nb = (blocks + parts - 1) / parts;
    k.share = 16 * nb;
    // as many workgroups as the registers were cut for, long-lived (8 rows, 32 updates, 25.6 M elements, 1 / 2 / 3 / 4 per unit: fp32 192 / 164 / 160 / 160 us)
    const int grid = (int)std::min<int64_t>(tiles, std::min(mma_waves(KS, nb) * num_cu, grid_cap));
    *grid_out = grid;
    const dim3 wg(grid, (k.U + k.share - 1) / k.share);
    switch (nb) {
#define X(N) case N: hipLaunchKernelGGL((norm_mma_kernel<KS, N, R>), wg, dim3(kBlock), 0, s, k, W); break;
        X(1) X(2) X(3) X(4)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <class R>
hipError_t launch_mma(WalkKernelArgs& k, int Wp, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    switch ((Wp + 3) / 4) {
#define X(N) \
    case N: return launch_mma_k<N, R>(k, Wp, num_cu, grid_cap, grid_out, s);
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace star
