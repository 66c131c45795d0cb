// gfx950 kernel for aggregation without the optimizer step: for every group u,
//     out_u[j] = sum_{w in G_u} c_{u,w} g_w[j]
// -- what a parent aggregates from its children and itself before it
// broadcasts in the all-reduce architecture (Section 4.2, "All-reduce
// architecture"), and what a tree node forwards upward (Section 4.4.2).
//
// Same layout and mapping as the update kernels: a thread owns chunks of 4
// elements, holds the W gradients of the chunk in registers, walks the groups
// with a wave-uniform member test (tables in LDS), fp32 FMA chain in ascending
// worker id.  Every row is read once, every output written once (fp32, or bf16
// rounded to nearest even).  Optional per-group norms as in the update kernel.
#include "star_device.h"

namespace star {

// The one group of a call, in the kernel arguments.
struct MeanArgs {
    void* out;
    uint32_t mask;
    float coef[STAR_MAX_WORKERS];
};

// LDS: out pointers [U] (8 bytes each) | coef[U][W] | mask[U] | (norms) wave[4][U] | nacc[U][kBlock]
template <int W, class R>
__global__ __launch_bounds__(kBlock) void reduce_rows_kernel(const RowPtrs rows, const float* __restrict__ t_coef,
                                                             const uint32_t* __restrict__ t_mask,
                                                             void* const* __restrict__ t_out, const int U,
                                                             const int out_bf16, const int64_t P, const int head,
                                                             const int norms, const int span_g, const int span_k,
                                                             double* __restrict__ partials,
                                                             const TileSource queue, const int claim,
                                                             const InlineTables inl) {
    extern __shared__ uint64_t lds64[];
    // out pointers | (norms) running sums of gbar^2 per thread and group, and per wave, in double (the
    // tiles a thread sees depend on the queue; see the step-by-step kernel) | coefficients | masks
    uint64_t* s_out = lds64;
    double* s_nacc = reinterpret_cast<double*>(s_out + U);
    double* s_wave = s_nacc + (norms ? U * kBlock : 0);
    float* s_coef = reinterpret_cast<float*>(s_wave + (norms ? (kBlock / 64) * U : 0));
    uint32_t* s_mask = reinterpret_cast<uint32_t*>(s_coef + U * W);
    if (t_coef) {
        for (int i = threadIdx.x; i < U * W; i += kBlock) s_coef[i] = t_coef[i];
        for (int i = threadIdx.x; i < U; i += kBlock) {
            s_mask[i] = t_mask[i];
            s_out[i] = reinterpret_cast<uint64_t>(t_out[i]);
        }
    } else {  // small tables ride in the kernel arguments
        for (int i = threadIdx.x; i < U * W; i += kBlock) s_coef[i] = inl.coef[i];
        for (int i = threadIdx.x; i < U; i += kBlock) {
            s_mask[i] = inl.mask[i];
            s_out[i] = reinterpret_cast<uint64_t>(inl.out[i]);
        }
    }
    if (norms)
        for (int u = 0; u < U; ++u) s_nacc[u * kBlock + threadIdx.x] = 0.0;
    __syncthreads();

    const Span span = make_span(span_g, span_k);
    const int64_t nchunk = P / 4;

    // one pass over the groups for the element(s) held in g; `store` writes gbar of group u
    auto walk = [&](float (&g)[W][4], auto&& store) {
        for (int u = 0; u < U; ++u) {
            const uint32_t m = __builtin_amdgcn_readfirstlane(s_mask[u]);
            float gb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < W; ++w) {  // ascending worker id; the test is uniform over the wave
                if (m & (1u << w)) {
                    const float c = s_coef[u * W + w];
#pragma unroll
                    for (int k = 0; k < 4; ++k) gb[k] = __builtin_fmaf(c, g[w][k], gb[k]);
                }
            }
            if (norms) {
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) s = __builtin_fmaf(gb[k], gb[k], s);  // unused slots hold 0
                s_nacc[u * kBlock + threadIdx.x] += (double)s;
            }
            const uint64_t o = s_out[u];
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)o);
            const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(o >> 32));
            store(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), gb);
        }
    };

    auto process = [&](const int64_t c) {
        typename R::vec raw[W];
#pragma unroll
        for (int w = 0; w < W; ++w) raw[w] = R::load(rows.p[w], c);
        float g[W][4];
        static_for<0, W>([&](auto wc) {
            constexpr int Wi = decltype(wc)::value;
            static_for<0, 4>([&](auto kc) {
                constexpr int K = decltype(kc)::value;
                g[Wi][K] = R::template get<K>(raw[Wi]);
            });
        });
        walk(g, [&](void* out, const float (&gb)[4]) {
            const f32x4 x = {gb[0], gb[1], gb[2], gb[3]};
            publish_chunk(x, out, out_bf16, c);
        });
    };
    if (claim > 0) {   // tiles from the queue
        const int64_t ntile = (nchunk + kBlock - 1) / kBlock;
        for_each_claimed_tile(queue, ntile, claim, [&](const int64_t tile) {
            const int64_t c = tile * kBlock + threadIdx.x;
            if (c < nchunk) process(c);
        });
    } else {
        int64_t c = span.first;
        for (int k = 0; k < span.K && c < nchunk; ++k, c += span.step) process(c);
    }
    const int64_t nrest = rest_count(head, P, nchunk);
    int64_t r = span.first;
    for (int k = 0; k < span.K && r < nrest; ++k, r += span.step) {
        const int64_t j = rest_element(r, head, nchunk);
        float g[W][4];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            g[w][0] = R::load1(rows.p[w], j);
            g[w][1] = g[w][2] = g[w][3] = 0.0f;
        }
        walk(g, [&](void* out, const float (&gb)[4]) {
            publish_element(gb[0], out, out_bf16, j);
        });
    }

    if (norms) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        for (int u = 0; u < U; ++u) {
            const double s = wave_sum_to_lane63(s_nacc[u * kBlock + threadIdx.x]);
            if (lane == 63) s_wave[wave * U + u] = s;
        }
        __syncthreads();
        for (int u = threadIdx.x; u < U; u += kBlock) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < kBlock / 64; ++q) s += s_wave[q * U + u];
            partials[(int64_t)u * gridDim.x + blockIdx.x] = s;
        }
    }
}

// One group without norms on long shards: the mean, or any weighted sum, of its rows, kept in LDS and written in bursts (see Burst).  The
// arithmetic is that of reduce_rows_kernel to the bit; coefficients and mask stay in scalar registers.
template <int W, class R>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, 1)))
void mean_burst_kernel(const RowPtrs rows, const MeanArgs mean, const int out_bf16, const int64_t P, const int head,
                       const TileSource queue, const int claim, const uint32_t period) {
    constexpr int CAP = burst_tiles<1>(0);
    __shared__ BurstRoom<CAP, 1> room;
    Burst<CAP, 1> burst(room, period);
    typedef typename R::vec vec_t;
    const int64_t nchunk = P / 4, ntile = (nchunk + kBlock - 1) / kBlock;
    auto fetch = [&](const int64_t tile, vec_t (&g)[W]) {
        const int64_t c = tile * kBlock + threadIdx.x;
        if (c < nchunk) {
#pragma unroll
            for (int w = 0; w < W; ++w) g[w] = R::load(rows.p[w], c);
        }
    };
    auto write = [&](const int64_t tile, const f32x4 (&y)[1]) {
        if (tile * kBlock + threadIdx.x < nchunk) publish_through(y[0], mean.out, out_bf16, tile);
    };
    vec_t gn[W] = {};
    bool primed = false;
    for_each_claimed_tile_ahead(queue, ntile, claim, [&](const int64_t tile, const int64_t following) {
        if (!primed) {
            fetch(tile, gn);
            primed = true;
        }
        vec_t g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) g[w] = gn[w];
        if (following >= 0) fetch(following, gn);
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
        static_for<0, W>([&](auto wc) {   // ascending worker id
            constexpr int Wi = decltype(wc)::value;
            if (mean.mask & (1u << Wi)) {
                static_for<0, 4>([&](auto kc) {
                    constexpr int K = decltype(kc)::value;
                    x[K] = __builtin_fmaf(mean.coef[Wi], R::template get<K>(g[Wi]), x[K]);
                });
            }
        });
        burst.put(tile, {x}, write);
    });
    burst.flush(write);
    const int64_t nrest = rest_count(head, P, nchunk);
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < nrest; r += (int64_t)gridDim.x * kBlock) {
        const int64_t j = rest_element(r, head, nchunk);
        float x = 0.0f;
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (mean.mask & (1u << w)) x = __builtin_fmaf(mean.coef[w], R::load1(rows.p[w], j), x);
        publish_element(x, mean.out, out_bf16, j);
    }
}

namespace {

size_t reduce_lds_bytes(int W, int U, bool norms) {
    return sizeof(uint64_t) * (size_t)U + sizeof(float) * ((size_t)U * W + (size_t)U) +
           (norms ? sizeof(double) * ((size_t)(kBlock / 64) * U + (size_t)U * kBlock) : 0);
}

// Long-lived workgroups per compute unit of an aggregation with norms in fixed assignment.  Enough for about 64 KB of rows in
// flight, at least two (32 bf16 rows, 16 groups, 32 Mi elements: one per unit 1.72 ms, two 0.91), with two exceptions,
// from 1 to 4 per unit over 1-32 rows, 1-8 groups, three kinds of groups and 0.3-60 M elements on the same buffers.
//  - Bound by memory (one or two groups, long shards) fewer in flight are better, as for the updates.  fp32, from 16 tiles a unit
//    on: one with 8 and more rows for one group, 12 and more for two (30 M elements: one group of 8 / 24 rows 166 / 438 us, 178 /
//    458 with two; two groups of 20 rows 433 against 467; but 3 M, 8 rows 25.1 against 23.6, and 10 M, 7 rows 56.7 against 54.2).
//    Four and five rows, for which 64 KB would be four: two, with any groups (30 M, 4 rows, one / four groups 89 / 174 against
//    95 / 194; 3 M, four groups 27.2 against 25.4; three and six rows are level).  bf16, one group, from 64 tiles a unit on: two
//    (30 M, 8 / 12 rows 95 / 124 against 101 / 132; level at 10 M).
//  - Bound by the walk over the groups (bf16 rows: half the bytes, the same arithmetic) more hide it while the shard is short,
//    where the memory can still take them: six and more groups of up to 24 rows below 16 tiles a unit four (1 M, 8 groups of
//    16 rows 21.2 us, 25.1 with two), beyond that, of 16 and more rows, three (10 M, 8 groups of 16 / 28 rows 131 / 179 against 145 /
//    206, 30 M, of 24 472 against 509), up to 64 tiles a unit with six or seven (60 M, 6 groups of 24 rows 858 against 837); three
//    to five groups of 16 to 24 rows three, below 16 tiles a unit only (3 M, 4 groups of 20 42.8 against 46.6; 30 M, 4 of 20
//    326 against 315, 3 of 24 355 against 321).
int sum_workgroups(int W, bool f32, int U, int64_t P, int num_cu) {
    const int64_t tiles = P / (4 * kBlock);
    const bool from16 = tiles >= 16 * (int64_t)num_cu, from64 = tiles >= 64 * (int64_t)num_cu;
    const int wg_bytes = W * (f32 ? 16 : 8) * kBlock;
    const int rule = std::max(2, std::min(4, (64 * 1024 + wg_bytes - 1) / wg_bytes));
    if (f32) {
        if (!from16) return rule;
        if ((U == 1 && W >= 8) || (U == 2 && W >= 12)) return 1;
        return W == 4 || W == 5 ? 2 : rule;
    }
    if (U == 1) return from64 && W >= 8 ? 2 : rule;
    if (U >= 6 && W <= 24 && !from16) return 4;
    if (W >= 16 && (U >= 8 || (U >= 6 && !from64) || (U >= 3 && W <= 24 && !from16))) return 3;
    return rule;
}

template <int W, class R>
hipError_t launch_reduce_t(const ReduceArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    if constexpr (W >= 6) {
        if (a.burst) {
            if (a.U != 1 || a.norms || a.coef || !a.queue) return hipErrorInvalidValue;
            const int grid = (int)std::min<int64_t>(std::min(num_cu, grid_cap), std::max<int64_t>(1, tiles_of(a.P)));
            MeanArgs m;
            m.out = a.inl->out[0];
            m.mask = a.inl->mask[0];
            for (int w = 0; w < STAR_MAX_WORKERS; ++w) m.coef[w] = w < W ? a.inl->coef[w] : 0.0f;
            *grid_out = grid;
            hipLaunchKernelGGL((mean_burst_kernel<W, R>), dim3(grid), dim3(kBlock), 0, s, a.rows, m, a.out_dtype == STAR_BF16 ? 1 : 0,
                               a.P, a.head, tile_source(a.queue, a.done), a.burst,
                               burst_period(burst_tiles<1>(0), (W * (int)sizeof(typename R::vec) + 16) * kBlock, grid));
            const hipError_t e = hipGetLastError();
            if (e == hipSuccess && a.told) *a.told = queue_tells(a.done, grid, a.burst, tiles_of(a.P));
            return e;
        }
    }
    auto kern = reduce_rows_kernel<W, R>;
    const size_t lds = reduce_lds_bytes(W, a.U, a.norms != 0);
    const bool queued = a.queue;
    const Geometry g = queued ? queue_geometry(num_cu, grid_cap, queue_workgroups_per_cu(0, false),
                                               W * (int)sizeof(typename R::vec) + 16, Traffic::Reduce)
                              // (with norms: long-lived workgroups)
                              : pick_geometry(a.P, a.norms != 0, num_cu, grid_cap, 256, 1,
                                              sum_workgroups(W, std::is_same<R, RowF32>::value, a.U, a.P, num_cu));
    *grid_out = g.grid;
    const Finished done = a.norms ? Finished() : a.done;
    hipLaunchKernelGGL(kern, dim3(g.grid), dim3(kBlock), lds, s, a.rows, a.coef, a.mask, a.out, a.U,
                       a.out_dtype == STAR_BF16 ? 1 : 0, a.P, a.head, a.norms, g.span_g, g.span_k, a.partials,
                       tile_source(a.queue, done), g.claim, a.coef ? InlineTables() : *a.inl);
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess && a.told) *a.told = queued && queue_tells(done, g.grid, g.claim, tiles_of(a.P));
    return e;
}

}  // namespace

int reduce_max_updates(int Wp, bool norms) {
    const size_t budget = 60 * 1024;  // stay inside 64 KB of LDS per workgroup
    int u = 1;
    while (u < 256 && reduce_lds_bytes(Wp, u + 1, norms) <= budget) ++u;
    return u;
}

hipError_t launch_group_reduce(int Wp, int dtype, const ReduceArgs& a, int num_cu, int grid_cap, int* grid_out,
                               hipStream_t s) {
    if (a.U < 1 || a.U > reduce_max_updates(Wp, a.norms != 0)) return hipErrorInvalidValue;
    switch (Wp) {
#define X(N)                                                                                         \
    case N:                                                                                          \
        return dtype == STAR_F32 ? launch_reduce_t<N, RowF32>(a, num_cu, grid_cap, grid_out, s)      \
                                 : launch_reduce_t<N, RowBf16x4>(a, num_cu, grid_cap, grid_out, s);
        STAR_FOR_EACH_W(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace star
