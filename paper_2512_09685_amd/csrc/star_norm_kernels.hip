// gfx950 kernel: per-group norms from direct sums of gbar_u^2, no update.
//
// The caller asked for direct sums (rows that may be anti-correlated), the coefficients have both signs, or the shard
// is very short; see decide() in star_api.cpp.  The arithmetic is y_u + 1 multiply-adds per element and update,
// and with more than a few updates that is what bounds the pass: 8 fp32 rows, 32 updates of 4.5 members on average,
// 25.6 M elements need 4.5 G fp32 multiply-adds (0.12 ms of the vector ALUs) and 0.82 GB (0.12 ms).
//   - A thread holds 16 or 8 elements of every row, so that one member test (a scalar branch) covers as many
//     multiply-adds, and so does the sum kept per update.
//   - Coefficients and member masks are read with scalar loads, one wait per update.
//   - Four squares are added in fp32, everything beyond in double (eight lanes in fp32 first would be 64 to 128 squares:
//     the partial sums' error grows fivefold, and elements of 1.6e18 give an infinite norm instead of 9.2e18).  So that the double
//     additions cost little, four updates are added over the wave together by swapping halves and quarters of it
//     between registers; eight lanes per wave and update then add into a double LDS slot of their own: 256 bytes per update, so
//     up to 240 updates need one pass over the rows, and several workgroups fit on a compute unit to hide the loads.
// Measured at that size: 203 us (195 with the fp32 sums over eight lanes), 601 with the step-by-step kernel this replaced (one
// LDS slot per thread and update, hence two passes for 32 updates and two waves per SIMD; coefficients from LDS at their
// use; 4 elements per thread); calls of that size go to norm_mma_kernel now (norms_on_matrix_cores).  Light rows pay more: 4 / 1 rows, 32 updates 122 / 73 against 112 / 66 (403 / 256 by the step-by-step kernel).
#include "star_norm_mma.h"

namespace star {

// Chunks of 4 elements a thread holds of every row.  Two also with 17 to 32 rows, although only two waves (32 rows: one)
// then fit on a SIMD: a member test for 4 multiply-adds costs more than the third wave brings (20 rows, 5 M elements,
// 128 updates 417 against 921 us; 32 rows, 25.6 M elements, 16 updates 754 against 879).
constexpr int walk_chunks(int W) { return W <= 4 ? 4 : 2; }

// LDS: slots[U][kSlots], double
constexpr int kSlots = kBlock / 8;
template <int W, class R>
__global__ __launch_bounds__(kBlock) void norm_walk_kernel(const WalkKernelArgs args) {
    constexpr int KCH = walk_chunks(W), E = 4 * KCH;
    extern __shared__ double walk_lds[];
    const auto* const in = (const STAR_CONST WalkKernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    // this workgroup's share of the updates
    const int u0 = (int)blockIdx.y * args.share, U = min(args.U - u0, args.share);
    const STAR_CONST float* coef = (const STAR_CONST float*)args.coef;
    const STAR_CONST uint32_t* mask = (const STAR_CONST uint32_t*)args.mask;
    if (!args.coef) {
        coef = in->inl.coef;
        mask = in->inl.mask;
    }
    coef += u0 * W;
    mask += u0;
    double* const s_slot = walk_lds;
    for (int i = threadIdx.x; i < (U + 3) / 4 * 4 * kSlots; i += kBlock) s_slot[i] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Four updates are added over the wave together: rows of 16 lanes end with update (0, 2, 1, 3)[row], lanes 0 to 7 of a row
    // write one slot each.  The slots are private to the lane, and turned by the update: four neighbours fall on four bank groups.
    const int row = lane >> 4, turn = 2 * (row & 1) + row / 2;
    double* const my_slot = s_slot + turn * kSlots + 8 * ((wave + turn) & 3) + (lane & 7);
    const bool writes = (lane & 8) == 0;

    auto add_four = [&](const int u, double q) {
        q += dpp_take<0x128, 0xf>(q);   // row_ror:8
        if (writes)
            __hip_atomic_fetch_add(my_slot + u * kSlots, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto walk = [&](const float (&g)[E][W]) {
        double one = 0.0, two = 0.0;
        for (int u = 0; u < U; ++u) {
            const uint32_t m = mask[u];
            float c[W];
#pragma unroll
            for (int w = 0; w < W; ++w) c[w] = coef[u * W + w];
            // all of them requested here, one wait (the loads would otherwise move to their uses, one wait a member)
#pragma unroll
            for (int w = 0; w < W; ++w) asm volatile("" ::"s"(c[w]));
            float gb[E];
#pragma unroll
            for (int k = 0; k < E; ++k) gb[k] = 0.0f;
#pragma unroll
            for (int w = 0; w < W; ++w) {   // ascending worker id; the test is uniform over the wave
                if (__builtin_expect((m >> w) & 1u, 1)) {
#pragma unroll
                    for (int k = 0; k < E; ++k) gb[k] = __builtin_fmaf(c[w], g[k][w], gb[k]);
                }
            }
            double s[KCH];
#pragma unroll
            for (int j = 0; j < KCH; ++j) {   // four squares in fp32, in double from there on
                float sq = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) sq = __builtin_fmaf(gb[4 * j + k], gb[4 * j + k], sq);
                s[j] = (double)sq;
            }
#pragma unroll
            for (int d = 1; d < KCH; d *= 2)
#pragma unroll
                for (int j = 0; j + d < KCH; j += 2 * d) s[j] += s[j + d];
            if (!(u & 1)) {
                one = s[0];
                continue;
            }
            const double pair = swap_add<32>(one, s[0]);
            if (!(u & 2)) {
                two = pair;
                continue;
            }
            add_four(u & ~3, swap_add<16>(two, pair));
        }
        if (U & 1) {
            const double pair = swap_add<32>(one, 0.0);
            add_four(U & ~3, U & 2 ? swap_add<16>(two, pair) : swap_add<16>(pair, 0.0));
        } else if (U & 2) {
            add_four(U & ~3, swap_add<16>(two, 0.0));
        }
    };

    const int64_t P = args.P, nchunk = P / 4;
    const int64_t width = (int64_t)kBlock * KCH, ntile = (nchunk + width - 1) / width;
    auto process = [&](const int64_t tile) {
        const int64_t c0 = tile * width + threadIdx.x;
        if (c0 - lane >= nchunk) return;   // the whole wave is beyond the end
        typename R::vec raw[KCH][W];
        const bool whole = (tile + 1) * width <= nchunk;
        // the row pointers are fetched again for every tile: kept, they would push the walk's coefficients out of the
        // scalar registers with 20 and more rows
        const STAR_CONST WalkKernelArgs* a = in;
        asm volatile("" : "+s"(a));
#pragma unroll
        for (int j = 0; j < KCH; ++j) {
            const int64_t c = c0 + (int64_t)j * kBlock;
            if (whole) {
#pragma unroll
                for (int w = 0; w < W; ++w) raw[j][w] = R::load(a->rows.p[w], c);
            } else {
                // the last tile: lanes beyond the end read the last chunk and hold zeros (a test around every load would
                // have the wave wait for one before it asks for the next)
                const int64_t last = c < nchunk ? c : nchunk - 1;
#pragma unroll
                for (int w = 0; w < W; ++w) raw[j][w] = R::load(a->rows.p[w], last);
#pragma unroll
                for (int w = 0; w < W; ++w)
                    if (c >= nchunk) raw[j][w] = typename R::vec{};
            }
        }
        float g[E][W];
        static_for<0, KCH>([&](auto jc) {
            constexpr int J = decltype(jc)::value;
            static_for<0, W>([&](auto wc) {
                constexpr int Wi = decltype(wc)::value;
                static_for<0, 4>([&](auto kc) {
                    constexpr int K = decltype(kc)::value;
                    g[4 * J + K][Wi] = R::template get<K>(raw[J][Wi]);
                });
            });
        });
        walk(g);
    };
    int64_t tile = blockIdx.x;
    for (; tile < ntile; tile += gridDim.x) process(tile);
    // at most 66 elements: as long as a tile, for the workgroup whose turn it is (found without the division, whose 170 instructions
    // every workgroup would go through: 2 M elements, 1 / 3 rows, 64 updates 28.6 / 34.8 us, so 27.1 / 32.6)
    const int64_t nrest = rest_count(args.head, P, nchunk);
    if (tile == ntile && threadIdx.x - lane < nrest) {
        float g[E][W];
#pragma unroll
        for (int k = 0; k < E; ++k)
#pragma unroll
            for (int w = 0; w < W; ++w) g[k][w] = 0.0f;
        if (threadIdx.x < nrest) {
            const int64_t j = rest_element(threadIdx.x, args.head, nchunk);
#pragma unroll
            for (int w = 0; w < W; ++w) g[0][w] = R::load1(args.rows.p[w], j);
        }
        walk(g);
    }
    __syncthreads();
    for (int u = wave; u < U; u += kBlock / 64) {   // one wave per update
        const double s = wave_sum_to_lane63(lane < kSlots ? s_slot[u * kSlots + lane] : 0.0);
        if (lane == 63) args.partials[(int64_t)(u0 + u) * gridDim.x + blockIdx.x] = s;
    }
}

// A shard of fewer tiles than units: the updates are shared out as well, in fours.  There the walk is one chain of updates
// long (16 rows, 16 updates, 5000 / 100 000 elements: 15.1 / 15.3 us a call, 19.9 / 20.7 in one piece; 8 rows, 32 updates: 15.2
// against 23), and each share's rows come out of the caches.  Up to 16 rows two workgroups a unit, which take turns at
// waiting (0.3 M elements, 64 updates of 4 / 8 / 16 rows: 21.6 / 38.7 / 55.1 with one, 18.9 / 22.6 / 29.6 with two; 32 rows, 0.1 M: 34.0, 38.4).
//   The rest is as long as a tile and gets workgroups of its own where the units have room for them beside the tiles' shares; it takes
// none away from those (64 tiles of 2048 elements and a rest, 64 updates, 20 / 32 rows: 27.5 / 35.7 us; 30.5 / 39.1 where the rest counted as a tile).
void walk_shape(int W, int most, int num_cu, int64_t tiles, bool rest, int U, int* grid, int* share) {
    const int room = (W <= 16 ? 2 : 1) * num_cu;
    *grid = (int)std::min<int64_t>(std::max<int64_t>(tiles, 1), most);
    const int parts = std::max(1, std::min(room / *grid, (U + 3) / 4));
    *share = ((U + parts - 1) / parts + 3) / 4 * 4;
    const int shares = (U + *share - 1) / *share;
    if (rest && *grid == tiles && tiles < most && (tiles + 1) * shares <= room) ++*grid;
}

namespace {

size_t walk_lds_bytes(int U) { return sizeof(double) * (size_t)((U + 3) / 4 * 4) * kSlots; }

// Workgroups per compute unit.  Four hide the loads of streams bound by arithmetic (and of light rows, which keep little in
// flight).  Up to about eight updates of heavier rows the pass is bound by memory, where fewer requests in flight are better:
// two workgroups, and one from 13 fp32 rows on with up to four updates (one / two per unit against four, mean of 8 to 60 M
// elements: 8 fp32 rows, 4 / 8 updates 1.07 / 0.96, 1.35 / 0.97; 16 rows, 2 updates 0.96 / 0.98; 5 rows, 4 / 8 updates 1.32 / 0.95,
// 1.77 / 1.09; 3 rows, 1 update 1.72 / 1.12; 16 bf16 rows, 4 / 8 updates 1.31 / 0.95, 1.54 / 0.97; 8 bf16 rows, 4 updates 1.83 / 1.13;
// 24 bf16 rows, 4 updates 1.20 / 1.00).  With 32 rows only one fits at a time, and one that stays is ahead of four after
// each other for longer streams too (25.6 M, 16 updates: fp32 695 against 765 us, bf16 657 against 701), except with one or two
// updates of bf16 rows (8 M, 2 updates: 79 against 75).
int walk_workgroups_per_cu(int W, bool f32, int U) {
    if (W > 28) return f32 || U > 2 ? 1 : 4;
    if (U > 8) return 4;
    if (f32 && W >= 13 && U <= 4) return 1;
    return W >= (U <= 4 ? (f32 ? 4 : 13) : (f32 ? 6 : 16)) ? 2 : 4;
}

template <int W, class R>
hipError_t launch_walk_t(WalkKernelArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    // Long-lived workgroups sweep the shard together, for every stream: the work queue is behind even where one or two
    // updates leave the pass bound by memory (1 fp32 row, 25.6 M elements, 1 update: 22 against 39 us; 16 rows, 2
    // updates: 232 against 252; 4 rows, 100 M elements: 241 against 246).
    const int per_cu = walk_workgroups_per_cu(W, std::is_same<R, RowF32>::value, a.U);
    const int64_t tiles = (a.P / 4 + (int64_t)kBlock * walk_chunks(W) - 1) / ((int64_t)kBlock * walk_chunks(W));
    int grid = 0, share = 0;
    walk_shape(W, std::min(per_cu * num_cu, grid_cap), num_cu, tiles, rest_count(a.head, a.P, a.P / 4) > 0, a.U, &grid, &share);
    *grid_out = grid;
    a.share = share;
    hipLaunchKernelGGL((norm_walk_kernel<W, R>), dim3(grid, (a.U + share - 1) / share), dim3(kBlock),
                       walk_lds_bytes(std::min(a.U, share)), s, a);
    return hipGetLastError();
}

}  // namespace

// Whether the matrix cores take the call (norm_mma_kernel): by what either kernel takes on 30 M elements once its arithmetic
// bounds it, in us.  The walk pays for every update, every coefficient it loads and every member (fp32 rows, 4 / 8 / 13 of them, 128
// updates of half the rows: 486 / 822 / 1163; of two: 396 / 587 / 727), more from 14 rows on, where fewer waves fit (16 / 24: 1660 / 2483,
// 1378 / 1836), and with 32 rows, where one does (6002, 4522).  The matrix cores pay for 16 updates at a time, and for the blocks that even
// out the workgroups (80 updates: six, see launch_mma_k): fp32 rows by row groups of four (1 / 2 / 4 / 8 of them, 128 updates: 389, 622,
// 1065, 2074), bf16 rows hardly by those (332, 366, 448, 735).  Where memory bounds both they are level, so the rule is good there too.
//   Up to 4 rows the walk is better on long shards than its count says, so the line lies higher there.  bf16 rows, walk / matrix cores:
// 8 / 30 M, 1 row, 64 updates 55 / 152 against 58 / 172, 3 rows, 24 updates of 1.5 members 31 / 84 against 33 / 94, but 1.1 M, 1 row, 128 updates 49
// against 32; fp32 rows: 30 M, 4 rows, 64 updates of 1.5 members 212 against 226, 3 rows of 2 219 against 225, but 8 M 76 against 75 and
// 76 against 73.
//   Short shards (walk / matrix cores, us a call): 0.1 M elements, 32 updates of 4 / 8 / 16 fp32 rows 10.4 / 10.2 / 18.2 against 11.7 / 10.4 / 15.8, 0.3 M
// 12.8 / 14.0 / 23.0 against 12.6 / 14.0 / 20.8; bf16 rows, whose rest is fetched step by step, 0.3 M 12.7 / 14.7 / 21.9 against 14.4 / 15.2 / 23.2, 0.6 M 14.6 / 21.6 /
// 33.7 against 15.6 / 17.1 / 26.3.
//   Timed against the walk alone, 1 to 32 rows, 1 to 128 updates, groups of one or two and of half the rows: where the rule says so the matrix cores
// are ahead 2.2 / 1.43 / 1.38 / 1.29 times on the mean with fp32 rows (0.3 / 2 / 8 / 30 M elements), 1.83 / 1.57 / 2.03 / 2.01 times with bf16 rows
// (0.5 / 2 / 8 / 30 M), and nowhere more than 2 % behind.
bool norms_on_matrix_cores(int Wp, bool f32, int U, int members, int64_t P) {
    if (P < (f32 ? 1 << 17 : 1 << 19) * (Wp > 4 ? 1 : 2)) return false;
    double walk = Wp <= 13 ? U * (1.6 + 0.25 * Wp) + 0.6 * members : U * (1.6 + 0.45 * Wp) + 0.55 * members;
    if (Wp > 28 && U > 4) walk *= 1.8;
    const int groups = (Wp + 3) / 4, parts = ((U + 15) / 16 + 3) / 4;   // of up to four blocks each
    const int blocks = parts * (((U + 15) / 16 + parts - 1) / parts);
    if (f32) return walk > blocks * (22 + 28 * groups) * (Wp > 4 ? 1.0 : P < 16 << 20 ? 1.1 : 1.25);
    return walk > (15.0 + blocks * (26 + 4 * groups)) * (Wp > 4 || P < 4 << 20 ? 1.0 : 1.45);
}

int walk_max_updates() { return 60 * 1024 / (int)walk_lds_bytes(4) * 4; }   // stay inside 64 KB of LDS per workgroup

hipError_t launch_norm_walk(int Wp, int dtype, const SeqArgs& a, int num_cu, int grid_cap, int* grid_out,
                            hipStream_t s) {
    if (a.U < 1 || a.U > walk_max_updates()) return hipErrorInvalidValue;
    WalkKernelArgs k;
    k.rows = a.rows;
    k.coef = a.coef;
    k.mask = a.mask;
    k.partials = a.partials;
    k.P = a.P;
    k.U = a.U;
    k.share = 0;
    k.head = a.head;
    k.inl = a.coef ? InlineTables() : *a.inl;
    if (norms_on_matrix_cores(Wp, dtype == STAR_F32, a.U, a.members, a.P))
        return dtype == STAR_F32 ? launch_norm_mma_f32(k, Wp, num_cu, grid_cap, grid_out, s)
                                 : launch_norm_mma_bf16(k, Wp, num_cu, grid_cap, grid_out, s);
    switch (Wp) {
#define X(N)                                                                                      \
    case N:                                                                                       \
        return dtype == STAR_F32 ? launch_walk_t<N, RowF32>(k, num_cu, grid_cap, grid_out, s)     \
                                 : launch_walk_t<N, RowBf16x4>(k, num_cu, grid_cap, grid_out, s);
        STAR_FOR_EACH_W(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace star
