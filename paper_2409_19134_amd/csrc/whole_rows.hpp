// Short rows whole: one workgroup computes a (user, KV head) row's attention over all of its tokens - one owner's, or both
// owners' and their merge (Theorem 1) - so that a call is one launch, without chunk partials and without a closing kernel.
// What bounds it: with few rows latency - two scalar round trips to the row's addresses (0.7 us), the tiles at what one
// compute unit can take in (~40 bytes a cycle: 16 KB per 0.17 us), and the instructions of the epilogue, ~2 ns each for
// the wave that executes them, hence a thread per channel there; with many rows HBM.  Workgroups of up to twelve waves
// (three per SIMD) that share a row's steps out evenly, both owners' in one line: the old split of such calls into
// one-step workgroups spread better over idle compute units but needed a second launch to close.  Measured, split kernels /
// this one (us per call): fp32 1 user 128 + 16 tokens 8.5 / 4.9 (fused), bf16 32 users of 64-512 + 1-256 with the append
// 18.9 / 15.2, 256 such users 90.3 / 82.3 (5.5 TB/s), 256 users of 24-192 + 64 51.2 / 31.5; fp16 with 64 channels, 16 users
// as three calls 19.8 / 14.2.  When it pays is whole_rows_choice's rule (schedule.hpp).
#pragma once
#include <type_traits>

#include "combine.hpp"
#include "partial_mfma.hpp"

namespace spd {

// The kernel's static part of the LDS.  The slots' results follow it and are read and written 16 bytes at a time, so its
// size is a multiple of 16.
struct alignas(16) RowsShared {
    float2 ml[kRowsMaxWaves + 1][16];  // running max and sum of every slot
    int n0;                            // slots [0, n0) are owner 0's
    int extra;                         // whether the extra slot is used
};
static_assert(sizeof(RowsShared) % 16 == 0, "the dynamic part starts where this ends");

// Waves per workgroup whose slots (one more than waves), with the static part, fit the 64 KB a launch may ask for: all twelve
// but with many query heads per KV head (6 for 16 heads of 128 channels).
__host__ __device__ constexpr int rows_waves_that_fit(int D, int G)
{
    const size_t n = (64 * 1024 - sizeof(RowsShared)) / staging_bytes(D, 1, G) - 1;
    return n > (size_t)kRowsMaxWaves ? kRowsMaxWaves : (int)n;
}

// One owner's call as the kernel needs it.
struct RowsOwner {
    const RowItem *items;
    const char *k_pool, *v_pool;  // paged mode
    const char *const *k_ptrs, *const *v_ptrs;  // contiguous mode with device pointer tables, else nullptr
    const int32_t *block_table;   // paged mode
    int32_t max_blocks, page_shift;
    int64_t token_stride, block_stride;  // bytes
    const char *k_new, *v_new;    // KV append
    float *out, *lse;
    int32_t grow;                 // see OwnerArgs
};

struct RowsArgs {
    RowsOwner a0, a1;    // a1: a copy of a0 unless `both`
    const int32_t *order;  // [n_users] users in launch order, or nullptr
    const char *q;       // [U][Hq][D]
    int32_t waves, both;  // both: both owners' rows, merged into y; else a0's alone - merged too if y is given, with a_in / lse_in
    int32_t Hkv, Hq, G;
    uint32_t wave_mul;   // ceil(2^32 / waves): x / waves is the high word of x * wave_mul
    float scale_log2e;
    const float *a_in, *lse_in;  // the other owner's finished partials
    float *y, *lse, *w_in;       // the merge's results, or nullptr
};

__device__ __forceinline__ RowItem scalar_load_row(const RowItem *items, int idx, int grow)
{
    static_assert(sizeof(RowItem) == 32, "a row is read as five dwords of eight");
    const const_u32_ptr w = (const_u32_ptr)(uintptr_t)(items + idx);
    RowItem it;
    it.k_base = reinterpret_cast<const char *>(((uint64_t)w[1] << 32) | w[0]);
    it.v_base = reinterpret_cast<const char *>(((uint64_t)w[3] << 32) | w[2]);
    it.t_end = (int32_t)w[4] + grow;
    return it;
}

// sum[v] += weight of slot S * os[S][v] over the slots; owner 0's sums (slots [0, n0)) move to `first`.
template <int MAXS, int VEC, int S = 0>
__device__ __forceinline__ void weighted_slots(const float (&os)[MAXS][VEC], float w, int n0, float (&first)[VEC], float (&sum)[VEC])
{
    if constexpr (S < MAXS) {
        if (S == n0) {  // uniform
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                first[v] = sum[v];
                sum[v] = 0.f;
            }
        }
        const float ws = row_dpp<0x150 + S>(w);  // row_newbcast: lane S's value
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            sum[v] = fmaf(ws, os[S][v], sum[v]);
        weighted_slots<MAXS, VEC, S + 1>(os, w, n0, first, sum);
    }
}

template <int VEC>
__device__ __forceinline__ void load_vec(float (&x)[VEC], const float *p)
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    const vec t = *reinterpret_cast<const vec *>(p);
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        x[v] = t[v];
}
template <int VEC>
__device__ __forceinline__ void store_vec(float *p, const float (&x)[VEC])
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    vec t;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        t[v] = x[v];
    *reinterpret_cast<vec *>(p) = t;
}

// Combines the slots' states and writes the row's results.  A thread takes VEC consecutive channels of one query head (one
// where the workgroup has a thread for every channel: this is the tail of a launch, and a wave's instructions take 2 ns
// each); the slots' weights are computed once per 16-lane row, lane i for slot i.  Straight-line over MAXS slots (the last
// one stands in, with weight 0, for those past n_slots), so that every LDS read leaves at once.  An owner's sums see its
// own slots only: a NaN in one owner's cache stays out of the other's partial.
template <int DT, int D, int MAXS, int VEC>
__device__ __forceinline__ void reduce_slots(const RowsArgs &A, const float2 (*sm_ml)[16], const float *sm_o, int n0, int n_slots,
                                             bool any0, bool any1, int64_t head0)
{
    constexpr int kOStride = o_stride(D);
    const int G = A.G, slot = threadIdx.x & 15;
    for (int idx = (int)threadIdx.x * VEC; idx < G * D; idx += (int)blockDim.x * VEC) {  // whole 16-lane rows: D / VEC >= 16
        const int g = idx / D, ch = idx % D;
        const int64_t at = head0 * D + idx, at_l = head0 + g;
        float x0[VEC] = {}, l0 = -INFINITY;
        if (A.y && !A.both) {  // the other owner's finished partial
            load_vec<VEC>(x0, A.a_in + at);
            l0 = A.lse_in[at_l];
        }
        const float2 ml = slot < n_slots ? sm_ml[slot][g] : make_float2(-INFINITY, 0.f);
        float os[MAXS][VEC];
#pragma unroll
        for (int s = 0; s < MAXS; ++s)
            load_vec<VEC>(os[s], sm_o + (min(s, n_slots - 1) * G + g) * kOStride + ch);
        const bool mine0 = slot < n0;
        const float M0 = row_max(mine0 ? ml.x : -INFINITY), M1 = row_max(mine0 ? -INFINITY : ml.x);
        const float w = ml.y == 0.f ? 0.f : fast_exp2(ml.x - (mine0 ? M0 : M1));  // a slot without steps holds l = 0
        const float wl = w * ml.y;
        const float L0 = row_sum(mine0 ? wl : 0.f), L1 = row_sum(mine0 ? 0.f : wl);
        float o0[VEC] = {}, o1[VEC] = {};
        weighted_slots<MAXS, VEC>(os, w, n0, o0, o1);
        // an infinite value times a stand-in's weight of 0 is NaN: once more, over the slots that there are
        float nan_if_any = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            nan_if_any += o0[v] + o1[v];
        if (__any(nan_if_any != nan_if_any)) {
            float sums[2][VEC] = {};
#pragma unroll 1
            for (int s = 0; s < n_slots; ++s) {
                float x[VEC];
                load_vec<VEC>(x, sm_o + (s * G + g) * kOStride + ch);
                const float ws = __shfl(w, s, 16);
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    sums[0][v] = s < n0 ? fmaf(ws, x[v], sums[0][v]) : sums[0][v];
                    sums[1][v] = s < n0 ? sums[1][v] : fmaf(ws, x[v], sums[1][v]);
                }
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                o0[v] = sums[0][v];
                o1[v] = n0 >= MAXS ? sums[0][v] : sums[1][v];
            }
        }
        // an owner without tokens: A = 0, lse = -inf
        const float i0 = fast_rcp(L0), i1 = fast_rcp(L1);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            o0[v] = any0 ? (n0 >= MAXS ? o1[v] : o0[v]) * i0 : 0.f;
            o1[v] = any1 ? o1[v] * i1 : 0.f;
        }
        const float e0 = any0 ? (M0 + fast_log2(L0) - Elt<DT>::kPShift) * kLn2 : -INFINITY;
        const float e1 = any1 ? (M1 + fast_log2(L1) - Elt<DT>::kPShift) * kLn2 : -INFINITY;
        store_vec<VEC>(A.a0.out + at, o0);
        if (ch == 0)
            A.a0.lse[at_l] = e0;
        if (!A.y)
            continue;
        float w0, w1, ls_y, y[VEC];
        if (A.both) {
            store_vec<VEC>(A.a1.out + at, o1);
            if (ch == 0)
                A.a1.lse[at_l] = e1;
            merge_weights(e0, e1, w0, w1, ls_y);
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                y[v] = (w0 == 0.f ? 0.f : w0 * o0[v]) + (w1 == 0.f ? 0.f : w1 * o1[v]);
        } else {  // owner 0 is the public owner, merged with the delivered private partials
            merge_weights(l0, e0, w0, w1, ls_y);
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                y[v] = (w0 == 0.f ? 0.f : w0 * x0[v]) + (w1 == 0.f ? 0.f : w1 * o0[v]);
        }
        store_vec<VEC>(A.y + at, y);
        if (ch == 0) {
            A.lse[at_l] = ls_y;
            A.w_in[at_l] = w0;
        }
    }
}

// The steps of both owners, laid end to end, are shared out to the waves in equal contiguous runs.  At most one wave gets
// the end of owner 0's steps and the beginning of owner 1's: its second result goes to one extra slot.
template <int DT, int D, bool PAGED, bool APPEND>
__global__ __launch_bounds__(kRowsMaxWaves * 64, 3) void whole_rows_kernel(RowsArgs A)
{
    constexpr int RB = D * Elt<DT>::kBytes;
    constexpr int NA = step_tiles(RB), kTile = step_tokens(RB);
    constexpr bool kTwo = RB == 128;  // two steps in flight where a step is 8 KB
    constexpr bool kQuad = DT == kF32Quad;
    constexpr int CP = D / 16;
    constexpr int kOStride = o_stride(D);
    __shared__ RowsShared sm;
    extern __shared__ __align__(16) float sm_o[];  // [waves + 1][G][kOStride]

    const int kvh = blockIdx.x;
    const int user = A.order ? scalar_load_i32(A.order, blockIdx.y) : (int)blockIdx.y;
    const int row = user * A.Hkv + kvh, G = A.G;
    const RowItem i0 = scalar_load_row(A.a0.items, row, A.a0.grow), i1 = scalar_load_row(A.a1.items, row, A.a1.grow);
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6)), W = A.waves;

    LaneConst L;
    L.r = lane & 15;
    L.grp = lane >> 4;
    L.kt = kQuad ? L.grp : L.r >> 2;
    L.kc = kQuad ? L.r >> 2 : L.grp;
    const int head = kQuad ? L.r & (kQuadHeads - 1) : L.r;  // the query head of the lane's Q operand and results
    const int64_t head0 = (int64_t)user * A.Hq + (int64_t)kvh * G;
    u32x4 qB[RB / 64];  // (lanes past the last head take a copy of it; their results are not stored)
    const char *qrow = A.q + (head0 + min(head, G - 1)) * RB + L.kc * 16;
#pragma unroll
    for (int kk = 0; kk < RB / 64; ++kk)
        qB[kk] = *reinterpret_cast<const u32x4 *>(qrow + kk * 64);

    const int S0 = (unsigned)(i0.t_end + kTile - 1) / kTile;
    const int S1 = A.both ? (unsigned)(i1.t_end + kTile - 1) / kTile : 0;
    const unsigned total = S0 + S1;
    const int lo = __umulhi(total * wave, A.wave_mul);  // wave 0: 0
    const int hi = wave + 1 == W ? (int)total : (int)__umulhi(total * (wave + 1), A.wave_mul);

    if (lane == 0) {
        if (lo < S0 && S0 <= hi) {  // the wave that holds owner 0's last step
            sm.n0 = wave + 1;
            sm.extra = S0 < hi;
        } else if (S0 == 0 && wave == 0) {
            sm.n0 = sm.extra = 0;
        }
    }

    // one run per wave, two for the wave that crosses from owner 0 to owner 1; a wave without steps leaves an idle slot
#pragma unroll 1
    for (int own = lo < S0 ? 0 : 1; own < 2; ++own) {
        const bool second = own != 0;
        const int b = second ? max(lo, S0) - S0 : lo, e = second ? hi - S0 : min(hi, S0);
        float m = -INFINITY, l = 0.f;
        f32x4 acc[CP];
#pragma unroll
        for (int cc = 0; cc < CP; ++cc)
            acc[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (b < e) {
            const int t_end = second ? i1.t_end : i0.t_end, t_last = t_end - 1;
            L.token_stride = second ? A.a1.token_stride : A.a0.token_stride;
            L.k_base = second ? i1.k_base : i0.k_base;
            L.v_base = second ? i1.v_base : i0.v_base;
            if constexpr (PAGED) {
                L.block_stride = second ? A.a1.block_stride : A.a0.block_stride;
                L.page_shift = second ? A.a1.page_shift : A.a0.page_shift;
                L.page_mask = (1 << L.page_shift) - 1;
                L.k_base += reinterpret_cast<uintptr_t>(second ? A.a1.k_pool : A.a0.k_pool);
                L.v_base += reinterpret_cast<uintptr_t>(second ? A.a1.v_pool : A.a0.v_pool);
                L.bt_row = (second ? A.a1.block_table : A.a0.block_table) + (int64_t)user * (second ? A.a1.max_blocks : A.a0.max_blocks);
            } else {
                L.k_base += user_base(second ? A.a1.k_ptrs : A.a0.k_ptrs, user);
                L.v_base += user_base(second ? A.a1.v_ptrs : A.a0.v_ptrs, user);
            }
            L.k_new_row = L.v_new_row = nullptr;
            const char *k_new = second ? A.a1.k_new : A.a0.k_new, *v_new = second ? A.a1.v_new : A.a0.v_new;
            // KV append: the wave that holds the row's last token reads it from the caller's buffer, and copies it to the cache
            // (16 bytes per lane, K in the first lanes, V in the next).  Its copy is asked for before the first tile and stored
            // when that has been asked for too: nothing waits for it.
            constexpr int kRowLanes = RB / 16;
            const bool append = APPEND && k_new && e == (second ? S1 : S0);
            u32x4 new_piece;
            int new_page = 0;
            if (append) {
                L.k_new_row = k_new + (int64_t)row * RB;
                L.v_new_row = v_new + (int64_t)row * RB;
                if (PAGED)
                    new_page = scalar_load_i32(L.bt_row, t_last >> L.page_shift);
                if (lane < 2 * kRowLanes)
                    new_piece = *reinterpret_cast<const u32x4 *>((lane < kRowLanes ? L.k_new_row : L.v_new_row) + (lane % kRowLanes) * 16);
            }
            auto store_new_token = [&] {
                if (append && lane < 2 * kRowLanes) {
                    int64_t off = (int64_t)(PAGED ? (t_last & L.page_mask) : t_last) * L.token_stride + (lane % kRowLanes) * 16;
                    if (PAGED)
                        off += (int64_t)new_page * L.block_stride;
                    *reinterpret_cast<u32x4 *>(const_cast<char *>(lane < kRowLanes ? L.k_base : L.v_base) + off) = new_piece;
                }
            };
            int tb = b * kTile;
            const int tb_end = min(e * kTile, t_end);
            PagePair P = {0, 0};
            if (PAGED)
                P = load_pages(L, tb, t_last);
            if constexpr (!kTwo) {
                // the first step in front of the loop or in it: which of the two the compiler schedules better differs (append, 1
                // user of 400 + 100 tokens 7.4 / 8.0 us contiguous, 8.6 / 8.2 paged; without the append, tiny fp32 5.0 / 4.9)
                if constexpr (APPEND && !PAGED) {
                    TileRegs<RB, NA> T;
                    load_tile<RB, NA, PAGED, APPEND>(T, L, tb, t_last, P, kTile);
                    store_new_token();
                    for (;;) {
                        compute_tile<DT, D>(T, qB, tb, L.grp, t_end, A.scale_log2e, m, l, acc);
                        tb += kTile;
                        if (tb >= tb_end)
                            break;
                        load_tile<RB, NA, PAGED, APPEND>(T, L, tb, t_last, P, kTile);
                    }
                } else {
                    for (; tb < tb_end; tb += kTile) {
                        TileRegs<RB, NA> T;
                        load_tile<RB, NA, PAGED, APPEND>(T, L, tb, t_last, P, kTile);
                        if (APPEND && tb == b * kTile)
                            store_new_token();
                        compute_tile<DT, D>(T, qB, tb, L.grp, t_end, A.scale_log2e, m, l, acc);
                    }
                }
            } else {
                TileRegs<RB, NA> T0, T1;
                load_tile<RB, NA, PAGED, APPEND>(T0, L, tb, t_last, P, kTile);
                store_new_token();
                for (;;) {
                    const bool more1 = tb + kTile < tb_end;
                    if (more1)
                        load_tile<RB, NA, PAGED, APPEND>(T1, L, tb + kTile, t_last, P, kTile);
                    compute_tile<DT, D>(T0, qB, tb, L.grp, t_end, A.scale_log2e, m, l, acc);
                    if (!more1)
                        break;
                    tb += 2 * kTile;
                    const bool more2 = tb < tb_end;
                    if (more2)
                        load_tile<RB, NA, PAGED, APPEND>(T0, L, tb, t_last, P, kTile);
                    compute_tile<DT, D>(T1, qB, tb - kTile, L.grp, t_end, A.scale_log2e, m, l, acc);
                    if (!more2)
                        break;
                }
            }
        }
        // the run's state, unscaled: the reduction below weights it
        const int slot = second && lo < S0 ? W : wave;
        l = wave_xor_sum<16>(l);
        l = wave_xor_sum<32>(l);
        if (L.grp == 0) {  // (4x4 blocks: entries past head 3 are copies, never read)
            sm.ml[slot][L.r] = make_float2(m, l);
        }
        if constexpr (kQuad)
            reduce_scatter_groups<CP>(acc);
        if (head < G) {
            float *dst = &sm_o[(slot * G + head) * kOStride];
            const int row0 = kQuad ? (L.r & ~3) : L.grp * 4, cc0 = kQuad ? (L.grp >> 1) * (CP / 2) + (L.grp & 1) * (CP / 4) : 0;
            if constexpr (kQuad) {
#pragma unroll
                for (int cc = 0; cc < CP / 4; ++cc)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        dst[o_channel<RB, CP>(row0 + v, cc0 + cc)] = acc[cc][v];
            } else {  // four phases are four consecutive channels
#pragma unroll
                for (int cc = 0; cc < CP; cc += 4)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        *reinterpret_cast<f32x4 *>(dst + o_channel<RB, CP>(row0 + v, cc)) =
                            f32x4{acc[cc][v], acc[cc + 1][v], acc[cc + 2][v], acc[cc + 3][v]};
            }
        }
        if (hi <= S0)
            break;
    }
    __syncthreads();

    const int n0 = uniform(sm.n0), n_slots = W + uniform(sm.extra);
    const bool thread_per_channel = G * D <= (int)blockDim.x;
    auto reduce = [&](auto max_slots, auto vec) {
        reduce_slots<DT, D, decltype(max_slots)::value, decltype(vec)::value>(A, sm.ml, sm_o, n0, n_slots, S0 > 0, S1 > 0, head0);
    };
    constexpr std::integral_constant<int, 5> few;  // four waves
    constexpr std::integral_constant<int, kRowsMaxWaves + 1> most;
    constexpr std::integral_constant<int, 1> one;
    constexpr std::integral_constant<int, 4> four;
    if (n_slots <= few)
        thread_per_channel ? reduce(few, one) : reduce(few, four);
    else
        thread_per_channel ? reduce(most, one) : reduce(most, four);
}

}  // namespace spd
