// gfx950 kernels for the group-synchronous parameter update.
//
// Layout: every buffer is a flat array of P elements, cut into "chunks" of VEC
// consecutive elements.  A wave works on 64 consecutive chunks, so it reads 64
// consecutive 16-byte pieces of each row: whole cache lines, every byte used
// once.  Workgroups are mapped to chunks in "spans": G consecutive workgroups
// sweep one contiguous span of G*K tiles together (tile = 256 chunks), each
// taking every G-th tile, so that at any moment the running workgroups touch a
// narrow, advancing window of every row (DRAM pages stay open) while each
// workgroup still lives for K tiles (one norm reduction per K tiles).  Each
// gradient row, params and momentum are read once per call; params and
// momentum are written once.  All state of an element lives in registers
// between the load and the store.
//
// Two evaluations of the U updates of a call (Section 1 items (2), (4);
// Section 4.2 of the paper define the updates):
//   seq_kernel  walks the updates one by one with the W gradients of the
//               element held in registers; group tables sit in LDS.
//   aff_kernel  applies the U updates as one affine map of (p, v, g_0..g_W-1)
//               whose coefficients the host composed in double precision; on many rows
//               aff_once_kernel and aff_burst_kernel do, on short and on long shards.
// Per-group norms: seq_kernel accumulates gbar_u^2 per thread (LDS slots; direct norms
// without an update have a kernel of their own, star_norm_kernels.hip),
// aff_kernel accumulates the pairwise products of the rows (Gram matrix);
// both end with a wave64 DPP reduction and write one partial per block.
#include <hip/hip_runtime.h>

#include "star_device.h"

namespace star {

// ================================================================= affine kernel
template <int W>
__device__ __forceinline__ void gram_step(float (&acc)[W * (W + 1) / 2], const float (&g)[W]) {
    int e = 0;
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = a; b < W; ++b) {
            acc[e] = __builtin_fmaf(g[a], g[b], acc[e]);
            ++e;
        }
}

// What one workgroup does for a CoefCopy: requests 16 values a thread before it writes any (a read of the host's memory takes 1 to 2 us).
__device__ __forceinline__ void carry(const CoefCopy& copy) {
    for (int i0 = threadIdx.x; i0 < copy.n; i0 += 16 * kBlock) {
        double x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (i0 + k * kBlock < copy.n) x[k] = copy.src[i0 + k * kBlock];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (i0 + k * kBlock < copy.n) copy.dst[i0 + k * kBlock] = x[k];
    }
}

// KCH: chunks a thread loads together per tile when the tiles come from the queue (a tile is then
// KCH * 256 chunks).  More than one only for the Gram matrix alone on very few rows: a thread that loads 8
// to 32 bytes per tile keeps too little in flight (1 fp32 row: 0.40 of the HBM peak), whatever the claim.
template <int W, class R, bool UPDATE, bool GRAM, int KCH = 1>
__global__ __launch_bounds__(kBlock) void aff_kernel(float* __restrict__ params, float* __restrict__ momentum,
                                                     const RowPtrs rows, const AffCoef cf, const int64_t P,
                                                     const int head, const int span_g, const int span_k,
                                                     void* __restrict__ publish, const int publish_bf16,
                                                     double* __restrict__ partials, const TileSource queue,
                                                     const int claim, const CoefCopy copy) {
    // one workgroup more where the launch carries the norms' coefficients to device memory for gram_finish_kernel
    if constexpr (GRAM) {
        if (copy.n && (int)blockIdx.x == span_g) {
            carry(copy);
            return;
        }
    }
    constexpr int VEC = R::VEC;
    constexpr int NG = W * (W + 1) / 2;
    float acc[GRAM ? NG : 1];
#pragma unroll
    for (int e = 0; e < (GRAM ? NG : 1); ++e) acc[e] = 0.0f;
    // Second-level sums, one private LDS slot per thread and pair.  The register
    // accumulators are folded into them every kGramFold tiles, so no fp32 chain
    // of products is longer than 4*kGramFold terms: long chains of squares of
    // short-mantissa (bf16) values round down systematically, about 1e-9 per
    // term, because the low bits of a square are not uniformly distributed.
    // With few rows (up to kFewRows) there are few pairs: the slots are double and take the sums after
    // every chunk, which makes them independent of the order of the tiles (to 1e-16), so that this
    // variant can take its tiles from the queue like the plain one; and it has the registers for it.
    constexpr bool kFew = GRAM && gram_few_rows_form(W, std::is_same<R, RowF32>::value, UPDATE);
    typedef typename std::conditional<kFew, double, float>::type fold_t;
    __shared__ __align__(16) fold_t fold[GRAM ? NG * kBlock : 1];
    bool folded = kFew;   // the slots hold something (many rows: not before the first fold, on a short shard the last)
    if constexpr (kFew) {
#pragma unroll
        for (int e = 0; e < NG; ++e) fold[e * kBlock + threadIdx.x] = (fold_t)0;
    }
    auto fold_now = [&]() {
        if constexpr (GRAM) {
            if (folded) {
#pragma unroll
                for (int e = 0; e < NG; ++e) fold[e * kBlock + threadIdx.x] += (fold_t)acc[e];
            } else {
#pragma unroll
                for (int e = 0; e < NG; ++e) fold[e * kBlock + threadIdx.x] = (fold_t)acc[e];
                folded = true;
            }
#pragma unroll
            for (int e = 0; e < NG; ++e) acc[e] = 0.0f;
        }
    };

    const Span span = make_span(span_g, span_k);
    const int64_t nchunk = P / VEC;

    // one chunk: VEC elements of every row, the update, the pairwise products
    auto process = [&](const int64_t c) {
        typename R::vec g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) g[w] = R::load(rows.p[w], c);
        float pe[VEC], ve[VEC];
        if constexpr (UPDATE) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                const f32x4 pq = load_state(params, c * (VEC / 4) + q);
                const f32x4 vq = load_state(momentum, c * (VEC / 4) + q);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    pe[4 * q + k] = pq[k];
                    ve[4 * q + k] = vq[k];
                }
            }
        }
        static_for<0, VEC>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            float ge[W];
            static_for<0, W>([&](auto wc) {
                constexpr int Wi = decltype(wc)::value;
                ge[Wi] = R::template get<K>(g[Wi]);
            });
            if constexpr (UPDATE) aff_step<W>(pe[K], ve[K], ge, cf);
            if constexpr (GRAM) gram_step<W>(acc, ge);
        });
        if constexpr (UPDATE) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) {
                f32x4 pq = {pe[4 * q], pe[4 * q + 1], pe[4 * q + 2], pe[4 * q + 3]};
                f32x4 vq = {ve[4 * q], ve[4 * q + 1], ve[4 * q + 2], ve[4 * q + 3]};
                store_state(pq, params, c * (VEC / 4) + q);
                store_state(vq, momentum, c * (VEC / 4) + q);
                if (publish) publish_chunk(pq, publish, publish_bf16, c * (VEC / 4) + q);
            }
        }
    };
    bool queued = false;
    if constexpr (kFew || !GRAM) {
        // without the register-heavy Gram accumulators the kernel affords a second copy of the chunk
        // code: tiles from the queue for long shards, a fixed assignment for short ones (heavy rows have kernels of their own for
        // the two)
        if (claim > 0) {
            queued = true;
            if constexpr (KCH > 1) {
                static_assert(GRAM && !UPDATE, "several chunks per thread: Gram matrix alone");
                const int64_t width = (int64_t)kBlock * KCH;
                const int64_t ntile = (nchunk + width - 1) / width;
                for_each_claimed_tile(queue, ntile, claim, [&](const int64_t tile) {
                    typename R::vec g[KCH][W];
#pragma unroll
                    for (int j = 0; j < KCH; ++j) {   // all loads of the tile first
                        const int64_t c = tile * width + (int64_t)j * kBlock + threadIdx.x;
#pragma unroll
                        for (int w = 0; w < W; ++w) g[j][w] = c < nchunk ? R::load(rows.p[w], c) : typename R::vec{};
                    }
#pragma unroll
                    for (int j = 0; j < KCH; ++j) {   // a chunk beyond the end holds zeros and adds nothing
                        static_for<0, VEC>([&](auto kc) {
                            constexpr int K = decltype(kc)::value;
                            float ge[W];
                            static_for<0, W>([&](auto wc) {
                                constexpr int Wi = decltype(wc)::value;
                                ge[Wi] = R::template get<K>(g[j][Wi]);
                            });
                            gram_step<W>(acc, ge);
                        });
                        fold_now();   // per chunk, as with one chunk per tile: the sums do not depend on KCH
                    }
                });
            } else {
                const int64_t ntile = (nchunk + kBlock - 1) / kBlock;
                for_each_claimed_tile(queue, ntile, claim, [&](const int64_t tile) {
                    const int64_t c = tile * kBlock + threadIdx.x;
                    if (c < nchunk) {
                        process(c);
                        if constexpr (kFew) fold_now();
                    }
                });
            }
        }
    }
    if (!queued) {
        int64_t c = span.first;
        for (int k = 0; k < span.K && c < nchunk; ++k, c += span.step) {
            if constexpr (GRAM && !kFew) {
                if ((k & (kGramFold - 1)) == kGramFold - 1) fold_now();
            }
            process(c);
            if constexpr (kFew) fold_now();
        }
    }
    // elements not covered by whole chunks: same arithmetic, one element at a time
    const int64_t nrest = rest_count(head, P, nchunk);
    int64_t r = span.first;
    for (int k = 0; k < span.K && r < nrest; ++k, r += span.step) {
        const int64_t j = rest_element(r, head, nchunk);
        float ge[W];
#pragma unroll
        for (int w = 0; w < W; ++w) ge[w] = R::load1(rows.p[w], j);
        if constexpr (UPDATE) {
            float pe = params[j], ve = momentum[j];
            aff_step<W>(pe, ve, ge, cf);
            params[j] = pe;
            momentum[j] = ve;
            if (publish) publish_element(pe, publish, publish_bf16, j);
        }
        if constexpr (GRAM) gram_step<W>(acc, ge);
    }

    // The workgroup's sum of every entry, in double: a wave takes an entry, four threads' slots a lane.  (Every wave summing its own registers
    // entry by entry, unrolled, was code that a short shard's launch spent 2 us on: it runs once, and is fetched for that.)
    if constexpr (GRAM) {
        fold_now();
        __syncthreads();
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        constexpr int kEach = (NG + kBlock / 64 - 1) / (kBlock / 64), N = kEach < 5 ? kEach : 5;   // N at a time: their additions wait for each other
#pragma unroll 1
        for (int i = 0; i < kEach; i += N) {
            double s[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int e = min(wave + kBlock / 64 * (i + k), NG - 1);
                const fold_t* const slot = fold + e * kBlock + 4 * lane;
                s[k] = ((double)slot[0] + (double)slot[1]) + ((double)slot[2] + (double)slot[3]);
            }
#pragma unroll
            for (int k = 0; k < N; ++k) s[k] = wave_sum_to_lane63(s[k]);
            if (lane == 63) {
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const int e = wave + kBlock / 64 * (i + k);
                    if (i + k < kEach && e < NG) partials[(int64_t)e * span_g + blockIdx.x] = s[k];   // (span_g: the workgroups that have sums)
                }
            }
        }
    }
}

// The collapsed update without norms on short shards of heavy rows, a tile a workgroup.  Such a launch lasts little longer than a workgroup takes to
// read its arguments and then its rows, and 32 rows have 64 registers' worth of pointers and 68 coefficients, more than a wave has scalar
// registers: left to itself the compiler fetches all of them before the first row and keeps what does not fit in the lanes of a vector register
// (four to seven rounds of fetches one behind the other, 100 to 390 moves).  So the arguments are read where they lie, the coefficients
// when the rows have been requested.  0.63 M elements, aff_kernel (with / without the queue's code) -> this one: 24 / 28 / 32 bf16 rows 8.4 / 9.4 / 10.4
// and 8.7 / 9.8 / 11.0 -> 7.2 / 7.6 / 8.3 us, 24 / 32 fp32 rows 12.6 / 16.6 and 12.7 / 17.5 -> 11.1 / 14.6; 2 M, 32 bf16 / fp32 rows 28.8 / 51.7 and 29.3 / 51.6 -> 26.8 /
// 49.0; 10 to 16 rows 0.3 us ahead.
struct OnceArgs {
    float* params;
    float* momentum;
    RowPtrs rows;
    AffCoef cf;
    int64_t P;
    void* publish;           // device copy of the new params, or null
    int32_t publish_bf16;
    int32_t head;            // see rest_element
};
template <int W, class R>
__global__ __launch_bounds__(kBlock) void aff_once_kernel(const OnceArgs) {
    typedef const __attribute__((address_space(4))) OnceArgs* args_t;   // (its only argument: it lies where the segment begins)
    const args_t args = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    // The same address, of which the compiler does not know that it is: what is read there is not read before what stands above.
    auto from_now_on = [&]() {
        args_t a = args;
        asm volatile("" : "+s"(a)::"memory");
        return a;
    };
    auto coefficients = [](const args_t args) {
        AffCoef cf;
        cf.dp = args->cf.dp;
        cf.m01 = args->cf.m01;
        cf.m10 = args->cf.m10;
        cf.m11 = args->cf.m11;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            cf.b0[w] = args->cf.b0[w];
            cf.b1[w] = args->cf.b1[w];
        }
        return cf;
    };
    const int64_t nchunk = args->P / 4;
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c < nchunk) {
        typename R::vec g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) g[w] = R::load(args->rows.p[w], c);
        f32x4 p = load_state(args->params, c), v = load_state(args->momentum, c);
        const args_t then = from_now_on();
        const AffCoef cf = coefficients(then);
        static_for<0, 4>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            float ge[W];
            static_for<0, W>([&](auto wc) {
                constexpr int Wi = decltype(wc)::value;
                ge[Wi] = R::template get<K>(g[Wi]);
            });
            float pe = p[K], ve = v[K];
            aff_step<W>(pe, ve, ge, cf);
            p[K] = pe;
            v[K] = ve;
        });
        store_state(p, then->params, c);
        store_state(v, then->momentum, c);
        if (then->publish) publish_chunk(p, then->publish, then->publish_bf16, c);
    }
    // elements not covered by whole chunks: same arithmetic, one element at a time (at most 66, the first workgroup's)
    if (blockIdx.x != 0) return;
    const args_t rest = from_now_on();
    if ((int64_t)threadIdx.x < rest_count(rest->head, rest->P, nchunk)) {
        const int64_t j = rest_element(threadIdx.x, rest->head, nchunk);
        float ge[W];
#pragma unroll
        for (int w = 0; w < W; ++w) ge[w] = R::load1(rest->rows.p[w], j);
        float pe = rest->params[j], ve = rest->momentum[j];
        aff_step<W>(pe, ve, ge, coefficients(rest));
        rest->params[j] = pe;
        rest->momentum[j] = ve;
        if (rest->publish) publish_element(pe, rest->publish, rest->publish_bf16, j);
    }
}

// The collapsed update without norms on long shards of heavy rows: tiles from the queue, one tile of look-ahead, results kept in LDS and
// written in bursts (see Burst), for which a compute unit holds one workgroup.
template <int W, class R>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, 1)))
void aff_burst_kernel(float* __restrict__ params, float* __restrict__ momentum, const RowPtrs rows, const AffCoef cf,
                      const int64_t P, const int head, void* __restrict__ publish, const int publish_bf16,
                      const TileSource queue, const int claim, const uint32_t period) {
    constexpr int CAP = burst_tiles(0);
    __shared__ BurstRoom<CAP> room;
    Burst<CAP> burst(room, period);
    typedef typename R::vec vec_t;
    const int64_t nchunk = P / 4, ntile = (nchunk + kBlock - 1) / kBlock;
    auto fetch = [&](const int64_t tile, vec_t (&g)[W], f32x4& p, f32x4& v) {
        const int64_t c = tile * kBlock + threadIdx.x;
        if (c < nchunk) {
#pragma unroll
            for (int w = 0; w < W; ++w) g[w] = R::load(rows.p[w], c);
            p = load_state(params, c);
            v = load_state(momentum, c);
        }
    };
    auto write = [&](const int64_t tile, const f32x4 (&x)[2]) {
        const int64_t c = tile * kBlock + threadIdx.x;
        if (c < nchunk) {
            store_through(x[0], params + tile * (4 * kBlock), threadIdx.x * 16);
            store_through(x[1], momentum + tile * (4 * kBlock), threadIdx.x * 16);
            if (publish) publish_through(x[0], publish, publish_bf16, tile);
        }
    };
    vec_t gn[W] = {};
    f32x4 pn = {0, 0, 0, 0}, vn = {0, 0, 0, 0};
    bool primed = false;
    for_each_claimed_tile_ahead(queue, ntile, claim, [&](const int64_t tile, const int64_t following) {
        if (!primed) {
            fetch(tile, gn, pn, vn);
            primed = true;
        }
        vec_t g[W];
#pragma unroll
        for (int w = 0; w < W; ++w) g[w] = gn[w];
        f32x4 p = pn, v = vn;
        if (following >= 0) fetch(following, gn, pn, vn);
        static_for<0, 4>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            float ge[W];
            static_for<0, W>([&](auto wc) {
                constexpr int Wi = decltype(wc)::value;
                ge[Wi] = R::template get<K>(g[Wi]);
            });
            float pe = p[K], ve = v[K];
            aff_step<W>(pe, ve, ge, cf);
            p[K] = pe;
            v[K] = ve;
        });
        burst.put(tile, {p, v}, write);
    });
    burst.flush(write);
    // elements not covered by whole chunks: same arithmetic, one element at a time (at most 66, the first workgroup's)
    const int64_t nrest = rest_count(head, P, nchunk);
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < nrest; r += (int64_t)gridDim.x * kBlock) {
        const int64_t j = rest_element(r, head, nchunk);
        float ge[W];
#pragma unroll
        for (int w = 0; w < W; ++w) ge[w] = R::load1(rows.p[w], j);
        float pe = params[j], ve = momentum[j];
        aff_step<W>(pe, ve, ge, cf);
        params[j] = pe;
        momentum[j] = ve;
        if (publish) publish_element(pe, publish, publish_bf16, j);
    }
}

// ================================================================= step-by-step kernel
// LDS: (norms) nacc[U][kBlock] | wave_part[4][U], both double | coef[U][W] | lr[U] | mask[U]
// nacc holds one running sum of gbar^2 per thread and update.  It is double because the tiles a
// thread sees depend on the queue: each chunk's fp32 sum of four squares is formed in a fixed order,
// and added in double the order of the chunks matters only at 1e-16.
template <int W, bool UPDATE, bool NORMS>
__device__ __forceinline__ void seq_steps(float (&g)[W][4], float (&p)[4], float (&v)[4],
                                          const float* s_coef, const float* s_lr, const uint32_t* s_mask,
                                          double* s_nacc, const int U, const float mu, const float wd) {
    // Running compensation of p over the updates of a launch (Kahan): p moves by increments far smaller
    // than itself, and U plain roundings of p would add up like sqrt(U) half-ulps (U = 300: beyond 1e-6).
    // With the lost low part carried along, p ends within an ulp of the exactly accumulated value for any
    // U.  A single update keeps the plain fused step (nothing to carry).
    float lost[4] = {0.0f, 0.0f, 0.0f, 0.0f};
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
        if constexpr (NORMS) {
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) s = __builtin_fmaf(gb[k], gb[k], s);  // unused slots hold 0
            s_nacc[u * kBlock + threadIdx.x] += (double)s;
        }
        if constexpr (UPDATE) {
            const float lr = s_lr[u];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float d = __builtin_fmaf(wd, p[k], gb[k]);   // d = gbar + wd p
                v[k] = __builtin_fmaf(mu, v[k], d);                // v = mu v + d
                if (U == 1) {
                    p[k] = __builtin_fmaf(-lr, v[k], p[k]);        // p = p - lr v
                } else {
                    const float y = __builtin_fmaf(-lr, v[k], -lost[k]);   // the step, less what the last sum dropped
                    const float t = p[k] + y;
                    lost[k] = (t - p[k]) - y;
                    p[k] = t;
                }
            }
        }
    }
}

// COLLAPSED (with NORMS): the norms are accumulated update by update as usual, the update itself is
// applied once, as the affine map `cf` of the whole stream.  For wide fp32 rows with norms and a short stream:
// the Gram matrix of 17 to 32 fp32 rows costs 1536 matrix flops per element whatever the stream, the direct
// sums y_u + 1 multiply-adds per update.
template <int W, class R, bool NORMS, bool COLLAPSED = false>
__global__ __launch_bounds__(kBlock) void seq_kernel(float* __restrict__ params, float* __restrict__ momentum,
                                                     const RowPtrs rows, const float* __restrict__ t_coef,
                                                     const float* __restrict__ t_lr,
                                                     const uint32_t* __restrict__ t_mask, const int U,
                                                     const float mu, const float wd, const int64_t P,
                                                     const int head, const int span_g, const int span_k,
                                                     void* __restrict__ publish, const int publish_bf16,
                                                     double* __restrict__ partials, const TileSource queue,
                                                     const int claim, const InlineTables inl, const AffCoef cf) {
    static_assert(R::VEC == 4, "the step-by-step kernel works on 4-element chunks");
    static_assert(!COLLAPSED || NORMS, "the collapsed update rides on the norm walk");
    extern __shared__ double lds[];
    double* s_nacc = lds;
    double* s_wave = s_nacc + (NORMS ? U * kBlock : 0);
    float* s_coef = reinterpret_cast<float*>(s_wave + (NORMS ? (kBlock / 64) * U : 0));
    float* s_lr = s_coef + U * W;
    uint32_t* s_mask = reinterpret_cast<uint32_t*>(s_lr + U);
    if (t_coef) {
        for (int i = threadIdx.x; i < U * W; i += kBlock) s_coef[i] = t_coef[i];
        for (int i = threadIdx.x; i < U; i += kBlock) {
            s_lr[i] = t_lr[i];
            s_mask[i] = t_mask[i];
        }
    } else {  // small tables ride in the kernel arguments
        for (int i = threadIdx.x; i < U * W; i += kBlock) s_coef[i] = inl.coef[i];
        for (int i = threadIdx.x; i < U; i += kBlock) {
            s_lr[i] = inl.lr[i];
            s_mask[i] = inl.mask[i];
        }
    }
    if constexpr (NORMS)
        for (int u = 0; u < U; ++u) s_nacc[u * kBlock + threadIdx.x] = 0.0;
    __syncthreads();

    const Span span = make_span(span_g, span_k);
    const int64_t nchunk = P / 4;

    auto process = [&](const int64_t c) {
        typename R::vec raw[W];
#pragma unroll
        for (int w = 0; w < W; ++w) raw[w] = R::load(rows.p[w], c);
        f32x4 pv = load_state(params, c);
        f32x4 vv = load_state(momentum, c);
        float p[4], v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            p[k] = pv[k];
            v[k] = vv[k];
        }
        float g[W][4];
        static_for<0, W>([&](auto wc) {
            constexpr int Wi = decltype(wc)::value;
            static_for<0, 4>([&](auto kc) {
                constexpr int K = decltype(kc)::value;
                g[Wi][K] = R::template get<K>(raw[Wi]);
            });
        });
        if constexpr (COLLAPSED) {
            seq_steps<W, false, true>(g, p, v, s_coef, s_lr, s_mask, s_nacc, U, mu, wd);
            static_for<0, 4>([&](auto kc) {
                constexpr int K = decltype(kc)::value;
                float ge[W];
#pragma unroll
                for (int w = 0; w < W; ++w) ge[w] = g[w][K];
                aff_step<W>(p[K], v[K], ge, cf);
            });
        } else {
            seq_steps<W, true, NORMS>(g, p, v, s_coef, s_lr, s_mask, s_nacc, U, mu, wd);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pv[k] = p[k];
            vv[k] = v[k];
        }
        store_state(pv, params, c);
        store_state(vv, momentum, c);
        if (publish) publish_chunk(pv, publish, publish_bf16, c);
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
        float p[4] = {params[j], 0, 0, 0}, v[4] = {momentum[j], 0, 0, 0};
        if constexpr (COLLAPSED) {
            seq_steps<W, false, true>(g, p, v, s_coef, s_lr, s_mask, s_nacc, U, mu, wd);
            float ge[W];
#pragma unroll
            for (int w = 0; w < W; ++w) ge[w] = g[w][0];
            aff_step<W>(p[0], v[0], ge, cf);
        } else {
            seq_steps<W, true, NORMS>(g, p, v, s_coef, s_lr, s_mask, s_nacc, U, mu, wd);
        }
        params[j] = p[0];
        momentum[j] = v[0];
        if (publish) publish_element(p[0], publish, publish_bf16, j);
    }

    if constexpr (NORMS) {
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

// ================================================================= finishing kernels
// They last a few microseconds, nearly all of it latency: of the launch, of one read, of the ticket and the word (together 0.5 to 1 us of a call
// that is waited for, 0.3 us more while the last workgroup put the ticket back with a store).  A wave takes one sum of partials, so that a launch
// has a quarter of the workgroups that one sum a workgroup would need, and its tickets (one a workgroup, 12 ns each at one place) as many fewer.
constexpr int kWaves = kBlock / 64;
inline dim3 finishing_grid(int n) { return dim3((n + kWaves - 1) / kWaves); }

// The sum of one row of partials, in lane 63 of the wave: in a fixed order, up to 512 of them requested together.
__device__ __forceinline__ double sum_partials(const double* __restrict__ row, const int grid) {
    constexpr int N = 8;
    double s = 0.0;
    for (int b0 = threadIdx.x & 63; b0 < grid; b0 += 64 * N) {
        double x[N];
#pragma unroll
        for (int k = 0; k < N; ++k) x[k] = b0 + 64 * k < grid ? row[b0 + 64 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < N; ++k) s += x[k];
    }
    return wave_sum_to_lane63(s);
}

// The workgroup has read what it needed of the slot.
__device__ __forceinline__ void finished_all(const Finished& done) {
    if (!done.word) return;
    __syncthreads();
    if (threadIdx.x == 0) finished(done);
}

__global__ __launch_bounds__(kBlock) void reduce_kernel(const double* __restrict__ partials, const int n, const int grid,
                                                        double* __restrict__ sums_out,
                                                        float* __restrict__ sqrt_out, const Finished done) {
    const int e = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (e < n) {
        const double t = sum_partials(partials + (int64_t)e * grid, grid);
        if ((threadIdx.x & 63) == 63) {
            if (sums_out) sums_out[e] = t;
            if (sqrt_out) sqrt_out[e] = (float)sqrt(t);
        }
    }
    finished_all(done);
}

// One workgroup per update u: n_u^2 = sum over pairs (a <= b) of c_a c_b Gamma_ab (off-diagonal pairs twice), each thread one pair or
// three, then a fixed-order sum in double.  (A wave per update, for a quarter of the tickets, has three to nine pairs a lane one behind the
// other: 0.3 M elements, update with norms, a call that is waited for, 16 fp32 rows, 16 updates 31.7 against 30.2 us, 32 bf16 rows, 64 updates
// 44.0 against 42.2, back to back 18.2 against 16.9 and 26.0 against 23.7; 16 bf16 rows, 256 updates 39.3 against 39.8 and 23.1 level.)
__global__ __launch_bounds__(kBlock) void gram_norms_kernel(const double* __restrict__ gamma,
                                                            const double* __restrict__ coef, const int U,
                                                            const int W, float* __restrict__ norms_out,
                                                            const Finished done) {
    __shared__ double s_wave[kWaves];
    const int u = blockIdx.x;
    const double* c = coef + (int64_t)u * W;
    const int ng = W * (W + 1) / 2;
    double s = 0.0;
    for (int e = threadIdx.x; e < ng; e += kBlock) {
        const double g = gamma[e];   // requested together with the coefficients: one memory latency, not two
        int a = 0, rem = e;
        while (rem >= W - a) {
            rem -= W - a;
            ++a;
        }
        const int b = a + rem;
        const double ca = c[a], cb = c[b];
        // rows outside the group take no part: a non-finite entry of a worker that is not a member (0 * inf)
        // must not reach this group's norm
        if (ca == 0.0 || cb == 0.0) continue;
        const double t = ca * cb * g;
        s += (a == b) ? t : 2.0 * t;
    }
    s = wave_sum_to_lane63(s);
    if ((threadIdx.x & 63) == 63) s_wave[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 64) finished(done);   // everyone has its pairs (another wave than the one that ends the sum)
    // a tiny negative sum (rounding of a quadratic form that is zero) gives 0; a non-finite one stays
    // non-finite, so that a bad gradient report shows in the norms of the groups it is part of
    if (threadIdx.x == 0 && u < U) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) t += s_wave[q];
        norms_out[u] = (float)sqrt(t < 0.0 && t > -1e300 ? 0.0 : t);
    }
}

// Both finishing steps in one launch, for the Gram matrix of up to kFinishRows rows on a short shard, where a call is bound by its
// launches: the waves sum the entries as in reduce_kernel, the workgroup that arrives last forms the norms.  The coefficients
// (read from the host's memory by gram_norms_kernel) are in device memory: the launch before carried them there.
// Update with norms, two launches -> one: 0.3 M elements, 1 / 4 / 8 fp32 rows 18.3 / 18.5 / 20.3 -> 14.1 / 14.1 / 16.6 us a call, 1 M, 4 / 8 rows 18.7 / 20.7
// -> 15.5 / 19.5, 2 M, 8 rows 28.5 -> 27.1, 4 M, 4 rows 31.8 -> 31.8 (1 to 1.5 us of each by the shorter way to the stream's handle; with
// buffers that change from call to call 0.3 M, 8 rows 18.1 -> 16.0 to 17.5).
// (With a workgroup of this launch to carry the coefficients: 0.3 M alike, but 18.3 -> 18.7 on buffers that are not in the caches.)
// Not for more rows: those are more sums for the last workgroup, and a hand-over between workgroups costs as much as a launch on
// the device, only less on the host.
__global__ __launch_bounds__(kBlock) void gram_finish_kernel(const double* __restrict__ partials, const int grid, double* gamma,
                                                             const double* __restrict__ coef, const int U, const int W,
                                                             unsigned int* ticket, float* __restrict__ norms_out,
                                                             const Finished done) {
    __shared__ int s_last;
    __shared__ double s_gamma[kFinishRows * kFinishRows];
    const int u = threadIdx.x;
    double c[kFinishRows];   // requested with the partials, by every workgroup: any may be the last
#pragma unroll
    for (int w = 0; w < kFinishRows; ++w) c[w] = u < U && w < W ? coef[u * W + w] : 0.0;
    const int e = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (e < W * (W + 1) / 2) {
        const double t = sum_partials(partials + (int64_t)e * grid, grid);
        if ((threadIdx.x & 63) == 63) __hip_atomic_store(gamma + e, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the wave's sum has reached the memory that all units see
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    // (at device scope: whoever has the slot next may start before this launch's caches are written back)
    if (threadIdx.x == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // nobody else is left
    if (threadIdx.x < kFinishRows * kFinishRows) {
        const int a = threadIdx.x / kFinishRows, b = threadIdx.x % kFinishRows;
        s_gamma[threadIdx.x] = a <= b && b < W ? __hip_atomic_load(gamma + a * W - a * (a - 1) / 2 + (b - a), __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT)
                                               : 0.0;
    }
    __syncthreads();
    if (u < U) {
        double s = 0.0;
#pragma unroll
        for (int a = 0; a < kFinishRows; ++a)
#pragma unroll
            for (int b = a; b < kFinishRows; ++b) {
                const double cc = (a == b ? 1.0 : 2.0) * c[a] * c[b];
                // rows outside the group take no part (0 * inf), see gram_norms_kernel
                s += c[a] == 0.0 || c[b] == 0.0 ? 0.0 : cc * s_gamma[a * kFinishRows + b];
            }
        norms_out[u] = (float)sqrt(s < 0.0 && s > -1e300 ? 0.0 : s);
    }
    if (!done.word) return;
    __syncthreads();   // everyone has its coefficients
    if (threadIdx.x == 0) tell_behind(done.word, done.seq);
}

// The last launch of the Gram matrix: entry e = (i, j), i <= j < W, of the packed triangle over Wp >= W rows (the kernels' padded
// row count) summed over the workgroups' partials as reduce_kernel does it, and written to both of its places in the full
// W x W matrix (zeros from a grid of 0, an empty shard).  A launch of its own for the second half cost 4 us a call
// (0.3 M elements, 8 fp32 / 16 bf16 rows 17.0 / 16.4 -> 12.8 / 12.6 us a call, 3 M, 16 bf16 rows 24.9 -> 23.3, 25.6 M 130.9 -> 129.0).
__global__ __launch_bounds__(kBlock) void reduce_gram_kernel(const double* __restrict__ partials, const int grid,
                                                             const int Wp, const int W, double* __restrict__ out,
                                                             const Finished done) {
    int i = 0, rem = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (rem < W * (W + 1) / 2) {
        while (rem >= W - i) {
            rem -= W - i;
            ++i;
        }
        const int j = i + rem;
        const double t = sum_partials(partials + (int64_t)(i * Wp - i * (i - 1) / 2 + rem) * grid, grid);
        if ((threadIdx.x & 63) == 63) {
            out[i * W + j] = t;
            out[j * W + i] = t;
        }
    }
    finished_all(done);
}

__global__ __launch_bounds__(kBlock) void fill_kernel(float* __restrict__ dst, const int64_t n, const float value) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dst[i] = value;
}

// ================================================================= launchers
int padded_rows(int Wc) {
    if (Wc <= 16) return Wc < 1 ? 1 : Wc;
    return (Wc + 3) / 4 * 4;
}

namespace {

size_t seq_lds_bytes(int W, int U, bool norms) {
    return sizeof(float) * ((size_t)U * W + 2 * (size_t)U) +
           (norms ? sizeof(double) * ((size_t)(kBlock / 64) * U + (size_t)U * kBlock) : 0);
}

template <int W, class R, bool NORMS, bool COLLAPSED = false>
hipError_t launch_seq_t(const SeqArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    auto kern = seq_kernel<W, R, NORMS, COLLAPSED>;
    const size_t lds = seq_lds_bytes(W, a.U, NORMS);
    // one or two updates are bound by memory and take their tiles from the queue; longer streams are bound
    // by arithmetic and latency and keep the fixed assignment with as many waves as fit
    const int thread_bytes = W * (int)sizeof(typename R::vec) + 32;
    // the collapsed form does so little arithmetic per update that it is bound by memory for any stream it is used for
    const bool queued = a.queue && (COLLAPSED || seq_takes_queue(a.U));
    // (the collapsed form's norm walk -- LDS reads and a wave-uniform branch per row and update -- needs a second
    // workgroup per unit to hide under the memory time: 20 to 32 fp32 rows, 8 updates, 0.68-0.71 of the HBM peak with
    // two against 0.43-0.45 with one)
    const int per_cu = COLLAPSED ? 2 : queue_workgroups_per_cu(thread_bytes, true);
    // (a single update of fp32 rows with its norm is bound by memory alone and, off the short shards, is fastest with
    // one or two workgroups per unit instead of the two to four that 64 KB in flight ask for: 20 / 32 M elements, 1 row
    // 70 / 113 against 77 / 121 us, 2 rows 85 / 138 against 93 / 150, 4 rows 109 / 167 against 120 / 188; 12 M, 8 rows 106
    // against 109; 3 M elements: level or behind.  Three rows lie between: two up to 64 tiles a unit, 6 / 12 M 34.0 / 62.1 us
    // against 35.6 / 63.4 with one; one beyond, 20 / 30 M 100 / 145 against 101 / 151)
    int one_report = 0;
    if (NORMS && !COLLAPSED && std::is_same<R, RowF32>::value && a.U == 1) {
        const int64_t tiles = a.P / (4 * kBlock);
        if (tiles >= 16 * (int64_t)num_cu) one_report = W <= 2 || (W == 3 && tiles < 64 * (int64_t)num_cu) ? 2 : 1;
    }
    const Geometry g = queued ? queue_geometry(num_cu, grid_cap, per_cu, thread_bytes)
                              : one_report ? pick_geometry(a.P, NORMS, num_cu, grid_cap, 256, 1, one_report)
                              : pick_geometry(a.P, NORMS, num_cu, grid_cap, thread_bytes, 4,
                                              COLLAPSED ? 2 : 1);   // (short shards as well: 25-30 % faster with two)
    *grid_out = g.grid;
    const Finished done = NORMS ? Finished() : a.done;
    hipLaunchKernelGGL(kern, dim3(g.grid), dim3(kBlock), lds, s, a.params, a.momentum, a.rows, a.coef, a.lr, a.mask,
                       a.U, a.mu, a.wd, a.P, a.head, g.span_g, g.span_k, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0,
                       a.partials, tile_source(a.queue, done), g.claim, a.coef ? InlineTables() : *a.inl, a.cf ? *a.cf : AffCoef());
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess && a.told) *a.told = queued && queue_tells(done, g.grid, g.claim, tiles_of(a.P));
    return e;
}

template <int W, class R, bool UPDATE, bool GRAM>
hipError_t launch_aff_t(const AffArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    // the Gram matrix alone on very few rows: enough chunks per thread for about 64 bytes in flight
    constexpr int kRowBytes = W * (int)sizeof(typename R::vec);
    // (134 M elements, 1 / 2 / 3 fp32 rows: 0.69 / 0.78 / 0.79 of the HBM peak against 0.40 / 0.66 / 0.78 with one
    // chunk; 1 / 2 / 3 bf16 rows with 4 / 4 / 2 chunks: 0.44 / 0.66 / 0.65 against 0.22 / 0.36 / 0.48)
    constexpr int KCH = (GRAM && !UPDATE && W <= kFewRows && kRowBytes < 64)
                            ? (kRowBytes <= 8 ? 8 : (kRowBytes <= 16 ? 4 : 2)) : 1;
    const bool queued = aff_takes_queue(GRAM, W, std::is_same<R, RowF32>::value, UPDATE) && a.queue;   // (heavy rows without norms: a.burst)
    if constexpr (KCH > 1) {
        if (queued) {
            const int thread_bytes = kRowBytes * KCH;
            const Geometry g = queue_geometry(num_cu, grid_cap, 2, thread_bytes, Traffic::ReadOnly);
            *grid_out = g.grid;
            hipLaunchKernelGGL((aff_kernel<W, R, UPDATE, GRAM, KCH>), dim3(g.grid), dim3(kBlock), 0, s, a.params,
                               a.momentum, a.rows, a.cf, a.P, a.head, g.span_g, g.span_k, a.publish,
                               a.publish_dtype == STAR_BF16 ? 1 : 0, a.partials, TileSource{a.queue, nullptr, 0u}, g.claim, CoefCopy());
            return hipGetLastError();
        }
    }
    if constexpr (UPDATE && !GRAM && bursts(W, std::is_same<R, RowF32>::value)) {
        if (a.burst) {
            const int grid = (int)std::min<int64_t>(std::min(num_cu, grid_cap), std::max<int64_t>(1, tiles_of(a.P)));
            if (!a.queue) return hipErrorInvalidValue;
            *grid_out = grid;
            hipLaunchKernelGGL((aff_burst_kernel<W, R>), dim3(grid), dim3(kBlock), 0, s, a.params, a.momentum, a.rows, a.cf, a.P,
                               a.head, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0, tile_source(a.queue, a.done), a.burst,
                               burst_period(burst_tiles(0), (kRowBytes + 64 + copy_bytes(a)) * kBlock, grid));
            const hipError_t e = hipGetLastError();
            if (e == hipSuccess && a.told) *a.told = queue_tells(a.done, grid, a.burst, tiles_of(a.P));
            return e;
        }
        const int64_t tiles = std::max<int64_t>(1, tiles_of(a.P));
        if (tiles > 0x7fffffff) return hipErrorInvalidValue;
        const OnceArgs once = {a.params, a.momentum, a.rows, a.cf, a.P, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0, a.head};
        *grid_out = (int)tiles;
        hipLaunchKernelGGL((aff_once_kernel<W, R>), dim3((unsigned)tiles), dim3(kBlock), 0, s, once);
        return hipGetLastError();
    } else {
        auto kern = aff_kernel<W, R, UPDATE, GRAM>;
        // long shards without the Gram accumulators: long-lived workgroups, tiles from the queue
        const int thread_bytes = W * (int)sizeof(typename R::vec) + (UPDATE ? 32 : 0);
        Geometry g = queued ? queue_geometry(num_cu, grid_cap, queue_workgroups_per_cu(thread_bytes, UPDATE), thread_bytes,
                                             UPDATE ? Traffic::Update : Traffic::ReadOnly)
                            : pick_geometry(a.P, GRAM, num_cu, grid_cap, 256, 1,
                                            sum_workgroups_per_cu(thread_bytes, UPDATE, a.P, num_cu));
        if (a.copy.n && queued) return hipErrorInvalidValue;   // (every workgroup of a queue's launch takes tiles)
        const Finished done = GRAM ? Finished() : a.done;
        *grid_out = g.grid;
        hipLaunchKernelGGL(kern, dim3(g.grid + (GRAM && a.copy.n ? 1 : 0)), dim3(kBlock), 0, s, a.params, a.momentum, a.rows, a.cf, a.P, a.head,
                           g.span_g, g.span_k, a.publish, a.publish_dtype == STAR_BF16 ? 1 : 0, a.partials,
                           tile_source(a.queue, done), g.claim, a.copy);
        const hipError_t e = hipGetLastError();
        if (e == hipSuccess && a.told) *a.told = queued && queue_tells(done, g.grid, g.claim, tiles_of(a.P));
        return e;
    }
}

template <int W>
hipError_t launch_seq_w(int dtype, bool norms, const SeqArgs& a, int num_cu, int grid_cap, int* grid_out, hipStream_t s) {
    if (a.cf) {   // collapsed update with direct norms: built for wide fp32 rows only
        if constexpr (W > 16) {
            if (dtype == STAR_F32 && norms) return launch_seq_t<W, RowF32, true, true>(a, num_cu, grid_cap, grid_out, s);
        }
        return hipErrorInvalidValue;
    }
    if (dtype == STAR_F32)
        return norms ? launch_seq_t<W, RowF32, true>(a, num_cu, grid_cap, grid_out, s)
                     : launch_seq_t<W, RowF32, false>(a, num_cu, grid_cap, grid_out, s);
    return norms ? launch_seq_t<W, RowBf16x4, true>(a, num_cu, grid_cap, grid_out, s)
                 : launch_seq_t<W, RowBf16x4, false>(a, num_cu, grid_cap, grid_out, s);
}

template <int W>
hipError_t launch_aff_w(int dtype, bool update, bool gram, const AffArgs& a, int num_cu, int grid_cap,
                        int* grid_out, hipStream_t s) {
    if constexpr (W <= 16) {
        if (gram) {
            if (dtype == STAR_F32) {
                if (update) return launch_aff_t<W, RowF32, true, true>(a, num_cu, grid_cap, grid_out, s);
                return launch_aff_t<W, RowF32, false, true>(a, num_cu, grid_cap, grid_out, s);
            }
            if (update) return launch_aff_t<W, RowBf16x4, true, true>(a, num_cu, grid_cap, grid_out, s);
            return launch_aff_t<W, RowBf16x4, false, true>(a, num_cu, grid_cap, grid_out, s);
        }
    }
    if (gram || !update) return hipErrorInvalidValue;
    if (dtype == STAR_F32) return launch_aff_t<W, RowF32, true, false>(a, num_cu, grid_cap, grid_out, s);
    return launch_aff_t<W, RowBf16x4, true, false>(a, num_cu, grid_cap, grid_out, s);
}

}  // namespace

int seq_max_updates(int Wp, bool norms) {
    // stay inside 64 KB of LDS per workgroup
    const size_t budget = 60 * 1024;
    int u = 1;
    while (u < 256 && seq_lds_bytes(Wp, u + 1, norms) <= budget) ++u;
    return u;
}

hipError_t launch_seq(int Wp, int dtype, bool norms, const SeqArgs& a, int num_cu, int grid_cap, int* grid_out,
                      hipStream_t s) {
    if (a.U < 1 || a.U > seq_max_updates(Wp, norms)) return hipErrorInvalidValue;
    switch (Wp) {
#define X(N) case N: return launch_seq_w<N>(dtype, norms, a, num_cu, grid_cap, grid_out, s);
        STAR_FOR_EACH_W(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_affine(int Wp, int dtype, bool update, bool gram, const AffArgs& a, int num_cu, int grid_cap,
                         int* grid_out, hipStream_t s) {
    if (!update && !gram) return hipErrorInvalidValue;
    switch (Wp) {
#define X(N) case N: return launch_aff_w<N>(dtype, update, gram, a, num_cu, grid_cap, grid_out, s);
        STAR_FOR_EACH_W(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_reduce(const double* partials, int n_out, int grid, double* sums_out, float* sqrt_out,
                         const Finished& done, hipStream_t s) {
    if (n_out < 1) return hipSuccess;
    hipLaunchKernelGGL(reduce_kernel, finishing_grid(n_out), dim3(kBlock), 0, s, partials, n_out, grid, sums_out, sqrt_out, done);
    return hipGetLastError();
}

hipError_t launch_gram_norms(const double* gamma, const double* coef, int U, int Wp, float* norms_out,
                             const Finished& done, hipStream_t s) {
    if (U < 1) return hipSuccess;
    hipLaunchKernelGGL(gram_norms_kernel, dim3(U), dim3(kBlock), 0, s, gamma, coef, U, Wp,
                       norms_out, done);
    return hipGetLastError();
}

hipError_t launch_gram_finish(const double* partials, int grid, double* gamma, const double* coef, int U, int W,
                              unsigned int* ticket, float* norms_out, const Finished& done, hipStream_t s) {
    if (W < 1 || W > kFinishRows || U < 1 || U > kBlock) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gram_finish_kernel, finishing_grid(W * (W + 1) / 2), dim3(kBlock), 0, s, partials, grid, gamma, coef, U, W, ticket,
                       norms_out, done);
    return hipGetLastError();
}

hipError_t launch_reduce_gram(const double* partials, int grid, int Wp, int W, double* out, const Finished& done, hipStream_t s) {
    hipLaunchKernelGGL(reduce_gram_kernel, finishing_grid(W * (W + 1) / 2), dim3(kBlock), 0, s, partials, grid, Wp, W, out, done);
    return hipGetLastError();
}

hipError_t launch_fill(float* dst, int64_t n, float value, hipStream_t s) {
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, dst, n, value);
    return hipGetLastError();
}

}  // namespace star
