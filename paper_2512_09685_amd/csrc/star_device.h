// Device-side building blocks shared by the kernel files: row access, streaming
// stores, the wave64 sum, the workgroup-to-tile mapping and the launch geometry.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "star_kernels.h"

namespace star {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// The same as they lie in memory: element-aligned only.  The hardware takes global loads and stores of 8 and 16
// bytes at any address (unaligned access mode, the default of the ROCm runtime and of the compiler), so these
// types cost nothing where the address is aligned and need no second code path where it is not.
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));

// ---------------------------------------------------------------- row access
// A "row type" says how VEC consecutive gradient elements are fetched with one
// load and how element k is widened to fp32.
struct RowF32 {
    static constexpr int VEC = 4;
    typedef f32x4 vec;
    static __device__ __forceinline__ vec load(const void* row, int64_t chunk) {
        return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(row) + chunk);
    }
    template <int K>
    static __device__ __forceinline__ float get(const vec& x) { return x[K]; }
    static __device__ __forceinline__ float load1(const void* row, int64_t j) {
        return reinterpret_cast<const float*>(row)[j];
    }
};

// bf16 is the upper half of an fp32: widening is a shift (even element of a
// dword) or a mask (odd element); exact, infinities and NaNs carried over.
template <int K>
__device__ __forceinline__ float bf16_of(uint32_t dword) {
    return (K & 1) ? __uint_as_float(dword & 0xffff0000u) : __uint_as_float(dword << 16);
}

struct RowBf16x4 {
    static constexpr int VEC = 4;
    typedef u32x2 vec;
    static __device__ __forceinline__ vec load(const void* row, int64_t chunk) {
        return __builtin_nontemporal_load(reinterpret_cast<const u32x2_any*>(row) + chunk);
    }
    template <int K>
    static __device__ __forceinline__ float get(const vec& x) { return bf16_of<K>(x[K >> 1]); }
    static __device__ __forceinline__ float load1(const void* row, int64_t j) {
        return __uint_as_float((uint32_t) reinterpret_cast<const uint16_t*>(row)[j] << 16);
    }
};

// Streaming (non-temporal) 16-byte store.  The empty asm pins the value in
// vector registers at this point; without it the optimiser re-forms the store
// from the scalar results and the non-temporal hint is lost.
__device__ __forceinline__ void store_streaming(f32x4 x, f32x4_any* dst) {
    asm volatile("" : "+v"(x));
    __builtin_nontemporal_store(x, dst);
}

// Params / momentum access: streamed (non-temporal), worth ~6 % on the mixed read / read-modify-write
// traffic.  The hint does not keep a small shard from staying in the 256 MB Infinity Cache between
// calls: shards with params + momentum up to that size ran equally fast with and without it.
__device__ __forceinline__ f32x4 load_state(const float* base, int64_t idx4) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(base) + idx4);
}
__device__ __forceinline__ void store_state(f32x4 x, float* base, int64_t idx4) {
    store_streaming(x, reinterpret_cast<f32x4_any*>(base) + idx4);
}

// fp32 -> bf16, round to nearest even; NaN stays NaN (quiet bit forced).
__device__ __forceinline__ uint32_t bf16_bits_rne(float x) {
    uint32_t b = __float_as_uint(x);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (b >> 16) | 0x40u;
    b += 0x7fffu + ((b >> 16) & 1u);
    return b >> 16;
}

// Streaming store of 4 consecutive values as fp32 or as bf16 (chunk index c).
__device__ __forceinline__ void publish_chunk(f32x4 x, void* dst, int as_bf16, int64_t c) {
    if (as_bf16) {
        u32x2 packed;
        packed[0] = bf16_bits_rne(x[0]) | (bf16_bits_rne(x[1]) << 16);
        packed[1] = bf16_bits_rne(x[2]) | (bf16_bits_rne(x[3]) << 16);
        asm volatile("" : "+v"(packed));
        __builtin_nontemporal_store(packed, reinterpret_cast<u32x2_any*>(dst) + c);
    } else {
        store_streaming(x, reinterpret_cast<f32x4_any*>(dst) + c);
    }
}

__device__ __forceinline__ void publish_element(float x, void* dst, int as_bf16, int64_t j) {
    if (as_bf16)
        reinterpret_cast<uint16_t*>(dst)[j] = (uint16_t)bf16_bits_rne(x);
    else
        reinterpret_cast<float*>(dst)[j] = x;
}

// ---------------------------------------------------------------- wave64 sum
// Sum over the 64 lanes with data-parallel-primitive moves; the total lands in
// lane 63.  Stages: swap within pairs, within quads, mirror within 8, mirror
// within 16 (every lane of a 16-lane row now holds the row's sum), then lane 15
// of rows 0 and 2 is added into rows 1 and 3, and lane 31 into rows 2 and 3.
// The order of additions is fixed, so the result is reproducible.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_take(float x) {
    // lanes outside ROW_MASK, or whose source lane is invalid, read 0
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_sum_to_lane63(float x) {
    x += dpp_take<0xB1, 0xf>(x);   // quad_perm [1,0,3,2]
    x += dpp_take<0x4E, 0xf>(x);   // quad_perm [2,3,0,1]
    x += dpp_take<0x141, 0xf>(x);  // row_half_mirror
    x += dpp_take<0x140, 0xf>(x);  // row_mirror
    x += dpp_take<0x142, 0xa>(x);  // row_bcast:15 into rows 1, 3
    x += dpp_take<0x143, 0xc>(x);  // row_bcast:31 into rows 2, 3
    return x;
}

// The same in double (each move is done on the two halves of the value).  The norm sums take this
// one: which tiles a workgroup gets from the queue differs from run to run, and only sums that are
// carried in double from the per-tile level on come out the same in fp32 every time.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_take(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double wave_sum_to_lane63(double x) {
    x += dpp_take<0xB1, 0xf>(x);
    x += dpp_take<0x4E, 0xf>(x);
    x += dpp_take<0x141, 0xf>(x);
    x += dpp_take<0x140, 0xf>(x);
    x += dpp_take<0x142, 0xa>(x);
    x += dpp_take<0x143, 0xc>(x);
    return x;
}

// Rows of SPAN lanes: the odd rows of x change places with the even rows of y, then the two are added.  Even rows of the
// result hold x's row plus its odd neighbour, odd rows the same of y.
template <int SPAN>
__device__ __forceinline__ u32x2 swap_rows(const uint32_t x, const uint32_t y) {
    const auto s = SPAN == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                              : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return u32x2{s[0], s[1]};
}
template <int SPAN>
__device__ __forceinline__ float swap_add(const float x, const float y) {
    const u32x2 s = swap_rows<SPAN>(__float_as_uint(x), __float_as_uint(y));
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
template <int SPAN>
__device__ __forceinline__ double swap_add(const double x, const double y) {
    const u32x2 lo = swap_rows<SPAN>((uint32_t)__double2loint(x), (uint32_t)__double2loint(y));
    const u32x2 hi = swap_rows<SPAN>((uint32_t)__double2hiint(x), (uint32_t)__double2hiint(y));
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// ---------------------------------------------------------------- compile-time loops
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// ---------------------------------------------------------------- elements outside whole chunks
// The host advances every pointer past the first `head` (0 to 63) elements of the shard, where that puts the buffers
// on whole cache lines; a shard cut out of larger buffers at an odd element is then read like any other (8 bf16
// rows, 46 M elements from element 1 on, update with norms and bf16 copy: 272 us, 437 one element per lane).  Chunks of 4 follow from
// there; what they leave over -- `head` elements before the pointers, up to 3 behind the last chunk -- is worked on one
// element at a time: remainder r is element rest_element(r), r = 0 .. rest_count() - 1.
__host__ __device__ __forceinline__ int64_t rest_count(const int head, const int64_t P, const int64_t nchunk) {
    return head + (P - nchunk * 4);
}
__device__ __forceinline__ int64_t rest_element(const int64_t r, const int head, const int64_t nchunk) {
    return r < head ? r - head : nchunk * 4 + (r - head);
}

// ---------------------------------------------------------------- workgroup -> tile mapping
// Workgroup b handles items first, first+step, ... (at most K of them, below n).
struct Span {
    int64_t first, step;
    int32_t K;
};
__device__ __forceinline__ Span make_span(const int span_g, const int span_k) {
    const int64_t G = span_g;
    Span s;
    s.first = ((int64_t)(blockIdx.x / span_g) * G * span_k + (blockIdx.x % span_g)) * kBlock + threadIdx.x;
    s.step = G * kBlock;
    s.K = span_k;
    return s;
}

// Dynamic order: the workgroups of a launch take tiles 0, 1, 2, ... from a queue, `claim` consecutive
// tiles at a time, and call body(tile) for each (the whole workgroup together; body may synchronise).
// Compared with a fixed assignment this keeps the tiles in flight a dense, slowly advancing window
// even though compute units progress at different rates, and it balances the end of the kernel.
// The next claim is requested before the current one is worked on, so the atomic's latency (several
// microseconds when 256 workgroups share one counter) is hidden.  Every workgroup leaves after its
// first claim beyond the last tile and requests nothing after that, so the loop ends for any queue
// state; the last one to leave puts the queue back to zero.
// The first claim of a workgroup is known without asking the counter: workgroup b gets 1 + b % claim
// tiles, laid out one after the other; the counter hands out the tiles after those (`base` on).  The
// unequal first claims are deliberate.  With equal ones all workgroups start, finish and re-claim at
// the same moments, every wave of the chip then walks the rows in step, and that pattern, once set,
// persists through the kernel: the 32-row bf16 aggregation ran 70 % slower that way (2.77 against
// 1.63 ms).  A spread of up to two tile times at the start is enough to keep the requests mixed.
__device__ __forceinline__ FirstClaim first_claim(const int claim, const int64_t ntile) {
    return first_claim_of((int64_t)blockIdx.x, (int64_t)gridDim.x, claim, ntile);
}

// What a workgroup does that uses its launch's workspace slot no more (one thread; the queue's last one to leave knows without a ticket that it is).
// The last ticket puts the counter back by itself: nothing has to reach the memory before the word, for which whoever waits for the call waits.
__device__ __forceinline__ void tell(uint32_t* word, const uint32_t seq) {
    __hip_atomic_store(word, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void finished(const Finished& f) {
    if (!f.word) return;
    if (gridDim.x > 1 && atomicInc(f.ticket, gridDim.x - 1) + 1 != gridDim.x) return;
    tell(f.word, f.seq);
}
// The same behind stores to the slot.
__device__ __forceinline__ void tell_behind(uint32_t* word, const uint32_t seq) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // tickets and queue are back at zero
    tell(word, seq);
}
__device__ __forceinline__ void leave(const TileSource& src) {
    // this workgroup's claims have all returned (their values were used), so when the count reaches the grid size nobody touches
    // `next` any more
    const unsigned int left = atomicAdd(&src.queue->done, 1u);
    if (left + 1 == gridDim.x) {
        atomicExch(&src.queue->next, 0ull);
        atomicExch(&src.queue->done, 0u);
        if (src.word) tell_behind(src.word, src.seq);
    }
}

template <class Body>
__device__ __forceinline__ void for_each_claimed_tile(const TileSource& src, const int64_t ntile, const int claim,
                                                      Body&& body) {
    TileQueue* const q = src.queue;
    __shared__ unsigned long long s_first;
    const FirstClaim fc = first_claim(claim, ntile);
    const int step = claim < 0 ? -claim : claim;
    // When the first claims already cover the shard nobody asks the counter, and nobody has to put it
    // back: the same for every workgroup of the launch (base and ntile are).
    const bool counter = fc.base < (unsigned long long)ntile;
    unsigned long long nxt = 0;
    int64_t t0 = fc.t0;
    int n = fc.n;
    while (t0 < ntile) {
        if (counter && threadIdx.x == 0) nxt = fc.base + atomicAdd(&q->next, (unsigned long long)step);
        const int64_t t1 = t0 + n < ntile ? t0 + n : ntile;
        n = step;
        for (int64_t t = t0; t < t1; ++t) body(t);
        if (!counter) break;
        if (threadIdx.x == 0) s_first = nxt;
        __syncthreads();
        t0 = (int64_t)s_first;
        __syncthreads();   // everyone has read s_first before thread 0 writes it again
    }
    if (counter && threadIdx.x == 0) leave(src);
}

// The same order with one tile of look-ahead, for kernels that issue the loads of the following tile
// before they work on the current one: body(tile, following) with following < 0 at the end.  The
// start of the next claim is made known to the whole workgroup when it begins the last tile of the
// current claim, so the look-ahead also crosses claims.
// `body` takes a first argument as well, which of SETS sets of registers holds the tile (an integral constant; they take turns): the
// following tile's loads go to the next set, so that nothing has to be moved.
template <int SETS, class Body>
__device__ __forceinline__ void for_each_claimed_tile_ahead(const TileSource& src, const int64_t ntile,
                                                            const int claim, Body&& body) {
    static_assert(SETS == 1 || SETS == 2, "one set or two");
    TileQueue* const q = src.queue;
    __shared__ unsigned long long s_first;
    const FirstClaim fc = first_claim(claim, ntile);
    const int step = claim < 0 ? -claim : claim;
    const unsigned long long base = fc.base;
    const bool counter = base < (unsigned long long)ntile;   // see for_each_claimed_tile
    unsigned long long nxt = 0;
    int64_t cur = fc.t0, end = 0;
    auto after = [&](const int64_t tile) {
        int64_t following = tile + 1;
        if (following >= end) {   // last tile of this claim: where does the next one start?
            if (!counter) {
                following = -1;
            } else {
                if (threadIdx.x == 0) s_first = nxt;
                __syncthreads();
                following = (int64_t)s_first;
                __syncthreads();
                if (following < ntile) {
                    // no claim is requested once the end is known: nothing may touch the queue
                    // after this workgroup has reported that it left
                    if (threadIdx.x == 0) nxt = base + atomicAdd(&q->next, (unsigned long long)step);
                    end = following + step < ntile ? following + step : ntile;
                } else {
                    following = -1;
                }
            }
        }
        return following;
    };
    if (cur < ntile && fc.n > 0) {   // (an even split of fewer tiles than workgroups leaves some without)
        if (counter && threadIdx.x == 0) nxt = base + atomicAdd(&q->next, (unsigned long long)step);
        end = cur + fc.n < ntile ? cur + fc.n : ntile;
        for (;;) {
            int64_t following = after(cur);
            body(std::integral_constant<int, 0>{}, cur, following);
            if (following < 0) break;
            cur = following;
            if constexpr (SETS == 2) {
                following = after(cur);
                body(std::integral_constant<int, 1>{}, cur, following);
                if (following < 0) break;
                cur = following;
            }
        }
    }
    if (counter && threadIdx.x == 0) leave(src);
}
template <class Body>
__device__ __forceinline__ void for_each_claimed_tile_ahead(const TileSource& src, const int64_t ntile, const int claim, Body&& body) {
    for_each_claimed_tile_ahead<1>(src, ntile, claim, [&](auto, const int64_t tile, const int64_t following) { body(tile, following); });
}

// ---------------------------------------------------------------- writes in bursts
// A stream of reads slows down by more than the writes' share when writes are mixed into it: 16 fp32 rows and the state, 110 M
// elements, 6.1 TB/s where the reads alone reach 6.7, because the DRAM has to turn its bus round again and again.  So long-lived
// workgroups keep what they would write in LDS, and all of them write at the same moments, which they read off the clock that all
// units of the GPU share (s_memrealtime, 100 MHz): whoever finds after a tile that the next period has begun writes what it holds.
// Nobody waits for anybody; a workgroup that runs out of room writes at once.  A thread reads back only what it has stored itself, so
// no barrier is needed either.  The same rows 1 455 -> 1 282 us; without the clock, every workgroup writing when its room is full, 1 515.
constexpr int kLdsBytes = 160 * 1024;
// 16 bytes of every lane, to consecutive places from a wave-uniform address on, at device scope and without the non-temporal hint: written
// through the L2 into the memory-side cache, which takes a burst faster than the DRAM (16 fp32 rows, 110 M elements 1 282 us; with the
// non-temporal hint 1 315, and 1 405 where lines of the rows or of the state are still dirty in that cache from whoever wrote them,
// 1 330 this way; at the default scope 1 492).
__device__ __forceinline__ void store_through(const f32x4 x, float* wave_base, const int lane_bytes) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(wave_base, 0, 0x7fffffff, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), r, lane_bytes, 0, 16 /* sc1 */);
}
// The same of a tile's chunk as fp32 or, rounded, as bf16, into the array `dst`: an aggregate, or the new parameters' copy.  A copy that went
// out with the non-temporal hint and at default scope in the middle of a burst cost more than the burst gained (with norms, 16 bf16 rows,
// 340 M elements, bf16 / fp32 copy: 2 942 / 3 141 us, kernels that write as they go 2 802 / 2 898, this way 2 684 / 2 813; 12 rows, 150 M: 1 119 / 1 195, 1 052 /
// 1 088, 1 038 / 1 099; 16 fp32 rows, 110 M: 1 499 / 1 580, 1 528 / 1 538, 1 420 / 1 459; without norms, 10 fp32 rows, 40 M: 394 / 417, 375 / 384, 367 / 380, 32 bf16 rows,
// 138 M: 1 901 / 2 000, 1 884 / 1 880, 1 770 / 1 810; written at once, beside the reads: 3 050 / 3 072 of the first).
__device__ __forceinline__ void publish_through(const f32x4 x, void* dst, const int as_bf16, const int64_t tile) {
    if (as_bf16) {
        u32x2 packed;
        packed[0] = bf16_bits_rne(x[0]) | (bf16_bits_rne(x[1]) << 16);
        packed[1] = bf16_bits_rne(x[2]) | (bf16_bits_rne(x[3]) << 16);
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint16_t*>(dst) + tile * (4 * kBlock), 0, 0x7fffffff, 0x00027000);
        __builtin_amdgcn_raw_buffer_store_b64(packed, r, threadIdx.x * 8, 0, 16 /* sc1 */);
    } else {
        store_through(x, reinterpret_cast<float*>(dst) + tile * (4 * kBlock), threadIdx.x * 16);
    }
}

template <int CAP, int N = 2>
struct BurstRoom {   // in LDS: N times 16 bytes a thread of every tile
    f32x4 x[CAP][N][kBlock];
    int32_t tile[kBlock / 64][CAP];
};
template <int N>
struct BurstRoom<0, N> {};
// Tiles that fit beside `other` bytes of LDS.
template <int N = 2>
constexpr int burst_tiles(int other) {
    return (kLdsBytes - 64 - other) / (int)sizeof(BurstRoom<1, N>);
}

template <int CAP, int N = 2>
struct Burst {
    BurstRoom<CAP, N>& room;
    const uint32_t period;   // ticks
    uint32_t next;
    int held = 0;

    __device__ __forceinline__ Burst(BurstRoom<CAP, N>& r, const uint32_t ticks) : room(r), period(ticks) { next = boundary(clock()); }
    static __device__ __forceinline__ uint32_t clock() { return (uint32_t)__builtin_readsteadycounter(); }
    __device__ __forceinline__ uint32_t boundary(const uint32_t now) const { return (now / period + 1) * period; }

    // The results of one chunk of a tile (the whole wave together); write(tile, results ...) stores them.
    template <class Write>
    __device__ __forceinline__ void put(const int64_t tile, const f32x4 (&x)[N], Write&& write) {
#pragma unroll
        for (int i = 0; i < N; ++i) room.x[held][i][threadIdx.x] = x[i];
        room.tile[threadIdx.x >> 6][held] = (int32_t)tile;
        ++held;
        const uint32_t now = clock();
        const bool due = (int32_t)(now - next) >= 0;
        if (held == CAP || due) flush(write);
        if (due) next = boundary(now);
    }
    template <class Write>
    __device__ __forceinline__ void flush(Write&& write) {
        constexpr int T = 4;   // tiles read together
        for (int i = 0; i < held; i += T) {
            f32x4 x[T][N];
            int64_t t[T];
#pragma unroll
            for (int k = 0; k < T; ++k) {
                const int j = i + k < held ? i + k : held - 1;
#pragma unroll
                for (int q = 0; q < N; ++q) x[k][q] = room.x[j][q][threadIdx.x];
                t[k] = __builtin_amdgcn_readfirstlane(room.tile[threadIdx.x >> 6][j]);
            }
#pragma unroll
            for (int k = 0; k < T; ++k)
                if (i + k < held) write(t[k], x[k]);
        }
        held = 0;
    }
};
template <int N>
struct Burst<0, N> {   // a kernel that writes as it goes
    __device__ __forceinline__ Burst(BurstRoom<0, N>&, uint32_t) {}
};

// ---------------------------------------------------------------- the collapsed update of one element
constexpr int kGramFold = 64;  // tiles between folds of the pairwise-product accumulators (power of two)

template <int W>
__device__ __forceinline__ void aff_step(float& p, float& v, const float (&g)[W], const AffCoef& cf) {
    // increment of p first, one final add: p is perturbed by one rounding of p itself
    float inc = cf.dp * p;
    inc = __builtin_fmaf(cf.m01, v, inc);
    float nv = cf.m10 * p;
    nv = __builtin_fmaf(cf.m11, v, nv);
#pragma unroll
    for (int w = 0; w < W; ++w) {  // ascending worker id
        inc = __builtin_fmaf(cf.b0[w], g[w], inc);
        nv = __builtin_fmaf(cf.b1[w], g[w], nv);
    }
    p = p + inc;
    v = nv;
}

// ================================================================= host side of a launch
// Launch geometry: G workgroups per span, K tiles per workgroup, and the grid.
struct Geometry {
    int grid, span_g, span_k;
    int claim;   // > 0: tiles come from the queue, this many per claim; span_g / span_k then serve the ragged end only
};

// Fixed assignment of tiles (short shards, launches without a queue).  A kernel that ends with a per-workgroup norm
// reduction runs long-lived workgroups that sweep the shard as a single span; the others get one
// tile per workgroup, dispatched in address order.
// `thread_bytes`: bytes one thread has in flight per tile; long-lived workgroups are stacked on a compute unit
// (up to `max_per_cu`) until about 64 KB per unit are in flight, which light bf16 kernels need and heavy fp32
// ones already have with one workgroup; `min_per_cu` is for kernels that need a second workgroup per unit for
// their arithmetic rather than for their memory traffic.
inline Geometry pick_geometry(int64_t P, bool reduces, int num_cu, int grid_cap,
                              int thread_bytes = 256, int max_per_cu = 1, int min_per_cu = 1) {
    const int64_t tiles = std::max<int64_t>(1, (P / 4 + kBlock - 1) / kBlock);
    Geometry g;
    g.claim = 0;
    if (reduces) {
        const int wg_bytes = std::max(1, thread_bytes) * kBlock;
        const int bpc = std::max(min_per_cu, std::min(max_per_cu, (64 * 1024 + wg_bytes - 1) / wg_bytes));
        g.span_g = (int)std::min<int64_t>(std::min(num_cu * bpc, grid_cap), tiles);
        g.span_k = 0x7fffffff;
        g.grid = g.span_g;
    } else {
        const int64_t max_grid = 0x7fffffff;
        g.span_g = 1;
        g.span_k = (int)((tiles + max_grid - 1) / max_grid);   // 1 unless the shard is absurdly long
        g.grid = (int)((tiles + g.span_k - 1) / g.span_k);
    }
    return g;
}

// Long-lived workgroups per compute unit of the vector-register Gram kernel in fixed assignment.  One keeps enough in
// flight from about 96 bytes per thread and chunk on; lighter rows want more, without the state to write back
// up to four (norms alone, 16 M elements, 2 / 3 / 4 fp32 and 2 bf16 rows: 30 / 40 / 51 / 24 us, 45 / 51 / 58 / 44 with one; update with norms, 8 /
// 16 / 30 M elements, 1 fp32 row: 35 / 59 / 106 us, 40 / 68 / 118 with one; 2 bf16 rows: 36 / 61 against 44 / 72), heavier
// ones lose by it (16 M, 4 / 6 fp32 rows: 102 / 131 against 93 / 114).  On a shard of a few tiles per unit a second
// workgroup halves the longest chain of tiles (3 M elements, 4 / 6 fp32 rows: 25.8 / 32.3 against 28.7 / 34.2; 1 M, 8 rows: 22.3
// against 23.8, but at 3 M, 8 rows: 39.2 against 38.3).
// (Two chunks requested together by a thread instead: level on one row, 8-12 % behind on 3 and 4 fp32 rows.)
inline int sum_workgroups_per_cu(int thread_bytes, bool update, int64_t P, int num_cu) {
    const int64_t tiles = P / (4 * kBlock);
    const bool few_tiles = tiles <= 4 * (int64_t)num_cu || (thread_bytes <= 128 && tiles <= 12 * (int64_t)num_cu);
    const int light = update ? (thread_bytes <= 48 ? 2 : 1) : std::max(1, std::min(4, 128 / thread_bytes));
    return std::max(light, few_tiles ? 2 : 1);
}

// Geometry of a launch that takes its tiles from a queue: `per_cu` long-lived workgroups per compute unit.
// Measured on MI355X, fewer waves in flight are faster as long as they keep enough bytes in flight: kernels
// that read-modify-write the state want one workgroup per unit from about 128 bytes per thread and tile
// (1 > 2 > 3 > 4 by 2-4 % each step), lighter ones and the read-mostly aggregation want two.
inline int queue_workgroups_per_cu(int thread_bytes, bool writes_state) {
    return writes_state && thread_bytes >= 128 ? 1 : 2;
}
// `tiles`: whole tiles of the shard if the launcher knows them (an estimate will do: the kernel splits
// its own count).  Up to short_tiles_per_workgroup() tiles per workgroup the launch takes the short-shard
// form of the first claims (first_claim_of) and no more workgroups than tiles.  Where the queue's order
// starts to pay, measured on the matrix-core kernel (the one that is in queue order at every length):
//   update with norms   8 tiles per workgroup (16 fp32 rows, 1 Mi elements: 27 against 34 us; 16 tiles: equal
//                       with one workgroup per unit, 2-7 % behind with two; 32 tiles: 10 % behind);
//                       16 tiles when a thread moves less than 160 bytes per tile (4 to 12 bf16 rows,
//                       6 and 8 Mi elements: 5-16 % ahead of 8)
//   norms / Gram alone  a pure read: 48 tiles (12 to 24 Mi elements: 2-10 % ahead of the queue, 32 Mi
//                       and more: 1-3 % behind with 16 to 32 rows); 128 tiles up to 128 bytes per thread and
//                       tile (8 bf16 rows, 16 to 64 Mi elements: 7-15 % ahead)
inline int short_tiles_per_workgroup(int thread_bytes, Traffic traffic) {
    if (traffic == Traffic::ReadOnly) return thread_bytes <= 128 ? 128 : 48;
    return thread_bytes < 160 ? 16 : 8;
}
inline Geometry queue_geometry(int num_cu, int grid_cap, int per_cu, int thread_bytes,
                               Traffic traffic = Traffic::Update, int64_t tiles = -1) {
    Geometry g;
    g.grid = g.span_g = std::max(1, std::min(num_cu * per_cu, grid_cap));
    g.span_k = 0x7fffffff;
    g.claim = queue_claim(thread_bytes, traffic);
    if (tiles >= 0 && tiles <= (int64_t)g.grid * short_tiles_per_workgroup(thread_bytes, traffic)) {
        g.claim = -1;
        g.grid = g.span_g = (int)std::max<int64_t>(1, std::min<int64_t>(g.grid, tiles));
    }
    return g;
}

// The period of the bursts, in ticks of 10 ns: the share `fill` of the time in which `workgroups` fill `cap` tiles of LDS at 6.6 TB/s, so
// that the clock comes before the room runs out (from 0.5 to 0.9 of it 1 % apart: the longer the fewer turns, but also the more
// workgroups that are early).
inline uint32_t burst_period(int cap, int bytes_per_tile, int workgroups, double fill = 0.75) {
    const double ticks = fill * cap * (double)bytes_per_tile * workgroups / 66000.0;
    return ticks < 100.0 ? 100u : (uint32_t)ticks;
}

// Bytes of the new parameters' copy that a thread writes per tile.
inline int copy_bytes(const AffArgs& a) { return !a.publish ? 0 : (a.publish_dtype == STAR_BF16 ? 8 : 16); }

inline int64_t tiles_of(int64_t P) { return (P / 4 + kBlock - 1) / kBlock; }

// Whether the workgroups of a launch of `grid` ask the queue's counter, whose last one to leave writes the word (for_each_claimed_tile).
inline bool queue_tells(const Finished& done, int grid, int claim, int64_t tiles) {
    return done.word && claim > 0 && first_claim_of(0, grid, claim).base < (unsigned long long)tiles;
}

#define STAR_FOR_EACH_W(X)                                                                                    \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(20) X(24) X(28) \
    X(32)

}  // namespace star
