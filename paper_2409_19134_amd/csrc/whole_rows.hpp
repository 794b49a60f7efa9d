// Short rows whole: one workgroup computes a (user, KV head) row's attention over all of its tokens - one owner's, or both
// owners' and their merge (Theorem 1) - so that a call is one launch, without chunk partials and without a closing kernel.
// What bounds it: with few rows latency - a scalar round trip to the row's address and the arguments, the tiles at what one
// compute unit can take in (~40 bytes a cycle: 16 KB per 0.17 us; how fast a wave asks makes no difference, row addresses of one
// instruction instead of seven gained nothing), and the instructions of the epilogue, ~2 ns each for the wave that executes them; with
// many rows HBM.  Workgroups of up to twelve waves
// (three per SIMD) that share a row's steps out evenly, both owners' in one line: the old split of such calls into
// one-step workgroups spread better over idle compute units but needed a second launch to close.  Measured, split kernels /
// this one (us per call): fp32 1 user 128 + 16 tokens 8.5 / 4.6 (fused), bf16 32 users of 64-512 + 1-256 with the append
// 18.9 / 14.8, 256 such users 90.3 / 81.9 (5.5 TB/s), 256 users of 24-192 + 64 51.2 / 31.5; fp16 with 64 channels, 16 users
// as three calls 19.8 / 13.4.  When it pays is whole_rows_choice's rule (schedule.hpp).
#pragma once
#include <cstddef>
#include <type_traits>

#include "combine.hpp"
#include "partial_mfma.hpp"

namespace spd {

// The kernel's static part of the LDS.  The slots' results follow it and are read and written 16 bytes at a time, so its
// size is a multiple of 16.
struct alignas(16) RowsShared {
    float2 ml[kRowsMaxWaves + 1][16];  // running max and sum of every slot
};
static_assert(sizeof(RowsShared) % 16 == 0, "the dynamic part starts where this ends");

constexpr int kFewSlots = 5;  // of up to four waves and the crossing one's second

// Waves per workgroup whose slots (one more than waves), with the static part, fit the 64 KB a launch may ask for: all twelve
// but with many query heads per KV head (6 for 16 heads of 128 channels).
__host__ __device__ constexpr int rows_waves_that_fit(int D, int G)
{
    const size_t n = (64 * 1024 - sizeof(RowsShared)) / staging_bytes(D, 1, G) - 1;
    return n > (size_t)kRowsMaxWaves ? kRowsMaxWaves : (int)n;
}

// The instances of at most 128 registers, of which a SIMD holds four waves, have a form held to three (but for the append in pages).  Where
// a unit gets its rows one after the other, the longest first, fewer at a time balance better; where all are resident, or many more, the
// fourth wave's loads count.  It takes the launches of up to two rows a unit (one workgroup of eight waves at a time instead of two: which
// rows share a unit is not settled at the start) and, of fp32, those of up to four (three at a time) and all with both owners.  us per call,
// four / three: 52 users of 352-1411 + 1-171 tokens, 8 heads, bf16 with the append 24.8 / 22.7, 116 of 60-608 + 1-233, 4 KV heads, fp32
// 29.2 / 25.5, 57 of 58-589 + 1-182 23.0 / 21.4; the append in pages 18.9 / 22.8 (57 of 426-853).  Four waves a row: fp32 49 of 80-322 +
// 1-192, 16 KV heads 32.5 / 30.2, 256 of 41-411 + 1-67, 4 KV heads 30.6 / 28.4; but one owner's 256 of 95-119 25.7 / 27.8, 16 bits with the
// append, 118 of 16-85 + 1-191, 13.6 / 14.7, in pages 139 of 26-269 12.3 / 13.1.
constexpr bool rows_three_waves_form(int DT, int D, bool PAGED, bool APPEND)
{
    return D == 64 && (DT == SPD_F32 || DT == kF32Quad ? !APPEND : PAGED != APPEND);
}

// Where the results go (the whole call's arrays).
struct RowsResults {
    float *out0, *lse0, *out1, *lse1;  // out1: nullptr unless both owners are the launch's
    const float *a_in, *lse_in;        // the other owner's finished partials, nullptr unless they were delivered
    float *y, *lse, *w_in;             // y: nullptr if nothing is merged
};

// What a paged call needs of an owner besides.
struct RowsPaging {
    const char *k_pool, *v_pool;
    const int32_t *block_table;
    int32_t max_blocks, page_shift;
    int64_t block_stride;  // bytes
};

// What a row's address and its share of the waves need, as the launch hands it over: in parameters of their own (HeadWords), which
// arrive in scalar registers with the wave (kernel-argument preloading: up to 14 dwords, not out of a struct).  The row is then asked
// for by a wave's first instructions instead of behind a scalar round trip to the arguments (us per call: tiny fp32 4.77 / 4.58, fp16
// three calls of 16 users 13.71 / 13.44, 32 users with the append 14.97 / 14.81).  Index 0 and 1: the owners; what belongs to owner 1
// repeats owner 0's unless `both`.
struct RowsHead {
    const RowItem *items[2];
    const int32_t *order;  // [n_users] users in launch order, or nullptr
    const char *q;         // [U][Hq][D]
    int32_t Hkv, G;
    int32_t grow[2];       // see OwnerArgs
    int32_t waves, both;   // both: both owners' rows, merged into y; else the first's alone - merged too if partials were delivered
};

// The rest, in the order in which a wave needs it: a scalar load of the arguments misses once for every 64-byte line, and the lines of
// one batch of loads don't come at once.  The kernel's last parameter.
struct RowsArgs {
    uint32_t wave_mul;     // ceil(2^32 / waves): x / waves is the high word of x * wave_mul
    float scale_log2e;
    int64_t token_stride[2];  // bytes
    const char *const *k_ptrs[2], *const *v_ptrs[2];  // contiguous mode with device pointer tables, else nullptr
    const char *k_new[2], *v_new[2];  // KV append, or nullptr
    RowsResults results;
    RowsPaging paging[2];
};
constexpr int kRowsArgsAt = sizeof(RowsHead);  // in the kernel's arguments (the launch checks it against the kernel's own parameters)

__device__ __forceinline__ RowItem scalar_load_row(Address items, int idx, int grow)
{
    static_assert(sizeof(RowItem) == 32, "a row is read as eight dwords at once");
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    typedef const u32x8 __attribute__((address_space(4))) *const_u32x8_ptr;
    const u32x8 w = *(const_u32x8_ptr)(items + (int64_t)idx * sizeof(RowItem));
    RowItem it;
    it.k_base = reinterpret_cast<const char *>(((uint64_t)w[1] << 32) | w[0]);
    it.v_base = reinterpret_cast<const char *>(((uint64_t)w[3] << 32) | w[2]);
    it.t_end = (int32_t)w[4] + grow;
    return it;
}

// The same as the kernel reads it: pointers that arrive through memory are told to be global ones (else: flat stores).
typedef float __attribute__((address_space(1))) *global_f32_ptr;
struct DevResults {
    global_f32_ptr out0, lse0, out1, lse1, a_in, lse_in, y, lse, w_in;
};
__device__ __forceinline__ DevResults scalar_load_results(uintptr_t at)
{
    static_assert(sizeof(RowsResults) == 72 && (kRowsArgsAt + offsetof(RowsArgs, results)) % 8 == 0, "read as nine pointers");
    const const_u64_ptr p = (const_u64_ptr)at;
    return DevResults{(global_f32_ptr)p[0], (global_f32_ptr)p[1], (global_f32_ptr)p[2], (global_f32_ptr)p[3], (global_f32_ptr)p[4],
                      (global_f32_ptr)p[5], (global_f32_ptr)p[6], (global_f32_ptr)p[7], (global_f32_ptr)p[8]};
}

template <int VEC>
struct FloatVec {
    typedef float type __attribute__((ext_vector_type(VEC)));
    typedef type __attribute__((address_space(1))) *global_ptr;
};
template <int VEC>
__device__ __forceinline__ void load_vec(float (&x)[VEC], const float *p)
{
    const auto t = *reinterpret_cast<const typename FloatVec<VEC>::type *>(p);
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        x[v] = t[v];
}
template <int VEC>
__device__ __forceinline__ void load_vec(float (&x)[VEC], global_f32_ptr p)
{
    const auto t = *(typename FloatVec<VEC>::global_ptr)p;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        x[v] = t[v];
}
template <int VEC>
__device__ __forceinline__ void store_vec(global_f32_ptr p, const float (&x)[VEC])
{
    typename FloatVec<VEC>::type t;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        t[v] = x[v];
    *(typename FloatVec<VEC>::global_ptr)p = t;
}

// One owner's slots [first, first + n) as a lane reduces them: lane i of every 16-lane row holds the running max and sum of slot
// first + i, each lane VEC channels of all slots.  Every LDS read leaves at once, in groups of four slots (a uniform branch each; a
// read past the owner's slots repeats its last one, with weight 0), so rows of few slots pay for few.
template <int D, int VEC>
struct SlotSums {
    static constexpr int kMost = kRowsMaxWaves, kGroup = 4;  // an owner has a slot per wave at most
    static_assert(kMost % kGroup == 0 && kMost <= 16);
    float2 ml;
    float x[kMost][VEC];
    int n, lane;

    __device__ __forceinline__ void load(const float2 (*sm_ml)[16], const float *sm_o, int first, int n_, int G, int g, int ch, int tid)
    {
        n = n_;
        lane = tid & 15;
        const int last = max(n - 1, 0);
        ml = sm_ml[first + min(lane, last)][g];
        const float *o = sm_o + (first * G + g) * o_stride(D) + ch;
        const int slot = G * o_stride(D), last_slot = last * slot;
#pragma unroll
        for (int s0 = 0; s0 < kMost; s0 += kGroup)
            if (s0 < n) {
#pragma unroll
                for (int s = s0; s < s0 + kGroup; ++s)
                    load_vec<VEC>(x[s], o + min(s * slot, last_slot));
            }
    }

    // GUARD: slots past the owner's are left out instead of given a weight of 0
    template <bool GUARD, int S = 0>
    __device__ __forceinline__ void weighted(float w, float (&o)[VEC]) const
    {
        if constexpr (S < kMost) {
            if (S % kGroup == 0 && S >= n)
                return;
            const float ws = row_dpp<0x150 + S>(w);  // row_newbcast: lane S's value
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                o[v] = fmaf(ws, GUARD && S >= n ? 0.f : x[S][v], o[v]);
            weighted<GUARD, S + 1>(w, o);
        }
    }

    // The owner's A and lse; without tokens (any false) 0 and -inf.
    __device__ __forceinline__ void reduce(bool any, float p_shift, float (&a)[VEC], float &lse) const
    {
        const bool on = lane < n;
        const float m = on ? ml.x : -INFINITY, l = on ? ml.y : 0.f;
        const float M = row_max_ordered(m);
        const float w = l == 0.f ? 0.f : fast_exp2(m - M);  // a slot without steps holds l = 0
        const float L = row_sum(w * l);
        float o[VEC] = {};
        weighted<false>(w, o);
        // an infinite value times a stand-in's weight of 0 is NaN: once more, over the slots that there are
        float nan_if_any = o[0];
#pragma unroll
        for (int v = 1; v < VEC; ++v)
            nan_if_any += o[v];
        if (__any(nan_if_any != nan_if_any)) {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                o[v] = 0.f;
            weighted<true>(w, o);
        }
        const float inv = fast_rcp(L);
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            a[v] = any ? o[v] * inv : 0.f;
        lse = any ? (M + fast_log2(L) - p_shift) * kLn2 : -INFINITY;
    }
};

// Where a thread's channels of a row are: the row's first head, its first channel of the result arrays, the thread's channels behind that.
struct RowAt {
    int64_t head0, from;
    unsigned at, g;
    bool first;  // of its head's channels
};

template <int VEC>
__device__ __forceinline__ void store_partial(global_f32_ptr out, global_f32_ptr lse, const RowAt &p, const float (&o)[VEC], float e)
{
    store_vec<VEC>(out + p.from + p.at, o);
    if (p.first)
        (lse + p.head0)[p.g] = e;
}

// The merge of a (private) and b (public).
template <int VEC>
__device__ __forceinline__ void store_merged(const DevResults &R, const RowAt &p, const float (&a)[VEC], float la, const float (&b)[VEC], float lb)
{
    float wa, wb, ls, y[VEC];
    merge_weights(la, lb, wa, wb, ls);
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        y[v] = (wa == 0.f ? 0.f : wa * a[v]) + (wb == 0.f ? 0.f : wb * b[v]);
    store_vec<VEC>(R.y + p.from + p.at, y);
    if (p.first) {
        (R.lse + p.head0)[p.g] = ls;
        (R.w_in + p.head0)[p.g] = wa;
    }
}

// sum[v] += weight of slot S * x[S][v] over the slots; owner 0's sums (slots [0, n0)) move to `first`.
template <int N, int VEC, int S = 0>
__device__ __forceinline__ void weighted_slots(const float (&x)[N][VEC], float w, int n0, float (&first)[VEC], float (&sum)[VEC])
{
    if constexpr (S < N) {
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
            sum[v] = fmaf(ws, x[S][v], sum[v]);
        weighted_slots<N, VEC, S + 1>(x, w, n0, first, sum);
    }
}

// Combines the slots' states of a workgroup of up to four waves and writes the row's results: five slots at most, both owners' at once,
// straight-line (the last slot stands in, with weight 0, for those past the row's).  Such workgroups are the shortest rows' or share a
// compute unit with others, so instructions count whichever wave executes them; owner by owner in groups of four, as below, is up to
// eight slot reads, two exponentials and two passes over them (us per call, below / this: 256 users of 24-192 + 1-64 tokens, 64 channels
// 20.0 / 18.9, in 16-token pages 18.4 / 17.5, 128 channels 31.9 / 31.1, fp32 32.9 / 32.5; the below form with groups of one 20.4).
// VEC: channels of a thread, one where the workgroup has a thread for each.
template <int DT, int D, int VEC>
__device__ __forceinline__ void reduce_few_slots(const DevResults &R, const float2 (*sm_ml)[16], const float *sm_o, int64_t head0, int G,
                                                 int threads, int n0, int n, bool any0, bool any1)
{
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // (see reduce_slots)
    const int slot = tid & 15;
    for (int idx = tid * VEC; idx < G * D; idx += threads * VEC) {  // whole 16-lane rows: D / VEC >= 16
        const unsigned g = (unsigned)idx / D, ch = (unsigned)idx % D;
        const RowAt p = {head0, head0 * D, (unsigned)idx, g, ch == 0};
        float x0[VEC] = {}, l0 = -INFINITY;
        if (R.a_in) {  // the other owner's finished partial
            load_vec<VEC>(x0, R.a_in + p.from + p.at);
            l0 = (R.lse_in + head0)[g];
        }
        const float2 ml = slot < n ? sm_ml[slot][g] : make_float2(-INFINITY, 0.f);
        float x[kFewSlots][VEC];
#pragma unroll
        for (int s = 0; s < kFewSlots; ++s)
            load_vec<VEC>(x[s], sm_o + (min(s, n - 1) * G + g) * o_stride(D) + ch);
        const bool mine0 = slot < n0;
        const float M0 = row_max_ordered(mine0 ? ml.x : -INFINITY), M1 = row_max_ordered(mine0 ? -INFINITY : ml.x);
        const float w = ml.y == 0.f ? 0.f : fast_exp2(ml.x - (mine0 ? M0 : M1));  // a slot without steps holds l = 0
        const float wl = w * ml.y, L0 = row_sum(mine0 ? wl : 0.f), L1 = row_sum(mine0 ? 0.f : wl);
        float o0[VEC] = {}, o1[VEC] = {};
        weighted_slots<kFewSlots, VEC>(x, w, n0, o0, o1);  // (n0 < kFewSlots: owner 0's always move)
        // an infinite value times a stand-in's weight of 0 is NaN: once more, over the slots that there are
        float nan_if_any = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            nan_if_any += o0[v] + o1[v];
        if (__any(nan_if_any != nan_if_any)) {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                o0[v] = o1[v] = 0.f;
#pragma unroll 1
            for (int s = 0; s < n; ++s) {
                float xs[VEC];
                load_vec<VEC>(xs, sm_o + (s * G + g) * o_stride(D) + ch);
                const float ws = __shfl(w, s, 16);
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    o0[v] = s < n0 ? fmaf(ws, xs[v], o0[v]) : o0[v];
                    o1[v] = s < n0 ? o1[v] : fmaf(ws, xs[v], o1[v]);
                }
            }
        }
        // an owner without tokens: A = 0, lse = -inf
        const float i0 = fast_rcp(L0), i1 = fast_rcp(L1);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            o0[v] = any0 ? o0[v] * i0 : 0.f;
            o1[v] = any1 ? o1[v] * i1 : 0.f;
        }
        const float e0 = any0 ? (M0 + fast_log2(L0) - Elt<DT>::kPShift) * kLn2 : -INFINITY;
        const float e1 = any1 ? (M1 + fast_log2(L1) - Elt<DT>::kPShift) * kLn2 : -INFINITY;
        store_partial<VEC>(R.out0, R.lse0, p, o0, e0);
        if (!R.y)
            continue;
        if (R.out1) {
            store_partial<VEC>(R.out1, R.lse1, p, o1, e1);
            store_merged<VEC>(R, p, o0, e0, o1, e1);
        } else {  // owner 0 is the public owner, merged with the delivered private partials
            store_merged<VEC>(R, p, x0, l0, o0, e0);
        }
    }
}

// The same for more waves, owner by owner.  A thread takes VEC consecutive channels of one query head: this is the
// tail of a launch, in which a wave's instruction takes 2 ns and two waves of a SIMD take turns, so the channels are spread over four
// waves - one per SIMD - where the workgroup has more than four.  (A channel per thread of eight waves, both owners' sums formed over
// all slots, with the argument order of then: tiny fp32 4.95 / 4.77 us, three calls of 16 users 14.25 / 13.85, 32 users with the append
// 15.12 / 14.97.)  In both forms an owner's sums see its own slots only: a NaN in one owner's cache stays out of the other's partial.
template <int DT, int D, int VEC, bool ONE_PASS>
__device__ __forceinline__ void reduce_slots(const DevResults &R, const float2 (*sm_ml)[16], const float *sm_o, int64_t head0, int G,
                                             int threads, int n0, int n1, bool any0, bool any1)
{
    // (an opaque copy: what follows from the thread's index is computed here.  Held across the tiles it cost the 64-channel instances up to
    // 13 registers and with them a wave per SIMD: 256 users of 24-192 + 1-64 tokens in pages 19.9 us, with the copy 18.4, and contiguous
    // with the append 20.7 / 18.4.)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    auto body = [&](int idx) __attribute__((always_inline)) {
        asm("" : "+s"(n0), "+s"(n1));  // (what follows from them is computed where it is used, not in front of the loop)
        const unsigned g = (unsigned)idx / D, ch = (unsigned)idx % D;
        const RowAt p = {head0, head0 * D, (unsigned)idx, g, ch == 0};
        float x0[VEC] = {}, l0 = -INFINITY;
        if (R.a_in) {  // the other owner's finished partial
            load_vec<VEC>(x0, R.a_in + p.from + p.at);
            l0 = (R.lse_in + head0)[g];
        }
        SlotSums<D, VEC> s0, s1;
        s0.load(sm_ml, sm_o, 0, n0, G, g, ch, tid);
        if (R.out1)
            s1.load(sm_ml, sm_o, n0, n1, G, g, ch, tid);
        float o0[VEC], e0;
        s0.reduce(any0, Elt<DT>::kPShift, o0, e0);
        store_partial<VEC>(R.out0, R.lse0, p, o0, e0);
        if (!R.y)
            return;
        if (R.out1) {
            float o1[VEC], e1;
            s1.reduce(any1, Elt<DT>::kPShift, o1, e1);
            store_partial<VEC>(R.out1, R.lse1, p, o1, e1);
            store_merged<VEC>(R, p, o0, e0, o1, e1);
        } else {  // owner 0 is the public owner, merged with the delivered private partials
            store_merged<VEC>(R, p, x0, l0, o0, e0);
        }
    };
    int idx = tid * VEC;  // whole 16-lane rows: D / VEC >= 16
    if constexpr (ONE_PASS) {
        if (idx < G * D)
            body(idx);
    } else {
        for (; idx < G * D; idx += threads * VEC)
            body(idx);
    }
}

// The steps of both owners, laid end to end, are shared out to the waves in equal contiguous runs.  At most one wave gets
// the end of owner 0's steps and the beginning of owner 1's: its second result goes to one extra slot.
// CHANNELS: the head's, negative: three waves per SIMD at most (see rows_three_waves_form).
template <int DT, int CHANNELS, bool PAGED, bool APPEND>
__global__ __launch_bounds__(kRowsMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(3, CHANNELS < 0 ? 3 : 8))) void whole_rows_kernel(
    u32x8 head_a, u32x4 head_b, u32x2 head_c, RowsArgs A)  // see RowsHead
{
    constexpr int D = CHANNELS < 0 ? -CHANNELS : CHANNELS;
    const RowsHead H = head_of<RowsHead>(head_a, head_b, head_c);
    const int Hkv = H.Hkv, G = H.G, waves = H.waves;
    const bool both = H.both;
    const Address items0 = (Address)H.items[0], items1 = (Address)H.items[1], q = (Address)H.q;
    constexpr int RB = D * Elt<DT>::kBytes;
    constexpr int NA = step_tiles(RB), kTile = step_tokens(RB);
    constexpr bool kTwo = RB == 128;  // two steps in flight where a step is 8 KB
    constexpr bool kQuad = DT == kF32Quad;
    constexpr int CP = D / 16;
    constexpr int kOStride = o_stride(D);
    __shared__ RowsShared sm;
    extern __shared__ __align__(16) float sm_o[];  // [waves + 1][G][kOStride]

    const int kvh = blockIdx.x;
    int user = blockIdx.y;
    if (H.order) {
        user = scalar_load_i32(H.order, user);
        asm volatile("" : "+s"(user));  // (its wait belongs in here: behind the branch it would be every launch's, for all loads so far)
    }
    const int row = user * Hkv + kvh, W = waves;
    const RowItem i0 = scalar_load_row(items0, row, H.grow[0]), i1 = scalar_load_row(items1, row, H.grow[1]);
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));

    LaneConst L;
    L.r = lane & 15;
    L.grp = lane >> 4;
    L.kt = kQuad ? L.grp : L.r >> 2;
    L.kc = kQuad ? L.r >> 2 : L.grp;
    const int head = kQuad ? L.r & (kQuadHeads - 1) : L.r;  // the query head of the lane's Q operand and results
    const int64_t head0 = (int64_t)row * G;
    u32x4 qB[RB / 64];  // (lanes past the last head take a copy of it; their results are not stored)
    const Address qrow = q + (head0 + min(head, G - 1)) * RB + L.kc * 16;
#pragma unroll
    for (int kk = 0; kk < RB / 64; ++kk)
        qB[kk] = *(const u32x4 __attribute__((address_space(1))) *)(qrow + kk * 64);

    // One wait for the row and for what its tiles need of the arguments: the compiler otherwise asks for the addresses behind the lengths.
    // (Every line of the arguments that a row needs is asked for here: one that is first touched later costs its whole trip there, the
    // results' 0.3 us.  Owner 0's paging lies in the line of w_in, owner 1's in the next.)
    asm volatile("" ::"s"(i0.k_base), "s"(i0.v_base), "s"(i1.k_base), "s"(i1.v_base), "s"(A.token_stride[0]), "s"(A.token_stride[1]),
                 "s"(A.k_ptrs[0]), "s"(A.v_ptrs[0]), "s"(A.k_ptrs[1]), "s"(A.v_ptrs[1]), "s"(A.wave_mul), "s"(A.k_new[0]), "s"(A.results.out0),
                 "s"(A.results.w_in));
    if constexpr (PAGED)
        asm volatile("" ::"s"(A.paging[1].block_stride));
    const int S0 = (unsigned)(i0.t_end + kTile - 1) / kTile;
    const int S1 = both ? (unsigned)(i1.t_end + kTile - 1) / kTile : 0;
    const unsigned total = S0 + S1;
    const int lo = __umulhi(total * wave, A.wave_mul);  // wave 0: 0
    const int hi = wave + 1 == W ? (int)total : (int)__umulhi(total * (wave + 1), A.wave_mul);

    // Slots [0, n0) are owner 0's: up to the first wave whose run reaches its last step (lane i looks at wave i).  If that run goes on
    // into owner 1's steps, the extra slot is used.
    const int run_end = lane + 1 < W ? (int)__umulhi(total * (lane + 1), A.wave_mul) : (int)total;
    const int n0 = S0 ? (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(run_end >= S0)) + 1 : 0;
    const bool extra = S0 && ((__builtin_amdgcn_ballot_w64(run_end > S0) >> (n0 - 1)) & 1);

    auto args = [&]() __attribute__((always_inline)) {  // (opaque: what is read through it is read there)
        uintptr_t at = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(at));
        return at + kRowsArgsAt;
    };

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
            L.token_stride = second ? A.token_stride[1] : A.token_stride[0];
            L.k_base = second ? i1.k_base : i0.k_base;
            L.v_base = second ? i1.v_base : i0.v_base;
            if constexpr (PAGED) {
                // The run's owner's entry, at an address of its own.  Chosen field by field from either owner's, both owners' were held, and
                // some of them spilled, across the tiles, and their trips stood one behind the other in front of the page ids (with the
                // order of the loads below, us per call: 16 users of 64-512 + 1-256 tokens with the append 13.7 / 12.5, 10 of 64-384 +
                // 1-128 9.8 / 8.9, 256 of 64 channels 46.6 / 42.4).
                const auto pg = (const RowsPaging __attribute__((address_space(4))) *)(args() + offsetof(RowsArgs, paging) + (second ? sizeof(RowsPaging) : 0));
                L.block_stride = pg->block_stride;
                L.page_shift = pg->page_shift;
                L.page_mask = (1 << L.page_shift) - 1;
                L.k_base += reinterpret_cast<uintptr_t>(pg->k_pool);
                L.v_base += reinterpret_cast<uintptr_t>(pg->v_pool);
                L.bt_row = pg->block_table + (int64_t)user * pg->max_blocks;
            } else {
                L.k_base += user_base(second ? A.k_ptrs[1] : A.k_ptrs[0], user);
                L.v_base += user_base(second ? A.v_ptrs[1] : A.v_ptrs[0], user);
            }
            int tb = b * kTile;
            const int tb_end = min(e * kTile, t_end);
            PagePair P = {0, 0};
            if (PAGED)  // (before the append asks for its page, which is not waited for)
                P = load_pages(L, tb, t_last);
            L.k_new_row = L.v_new_row = nullptr;
            const char *k_new = second ? A.k_new[1] : A.k_new[0], *v_new = second ? A.v_new[1] : A.v_new[0];
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

    // The results' pointers are read here, next to the slots: scalar registers that hold them across the tiles are spilled, and a spill
    // is an instruction each way.  (In front of the barrier the slowest wave would wait for them.)
    const DevResults R = scalar_load_results(args() + offsetof(RowsArgs, results));
    const int n1 = W + extra - n0;
    auto few = [&](auto vec) __attribute__((always_inline)) {
        reduce_few_slots<DT, D, decltype(vec)::value>(R, sm.ml, sm_o, head0, G, W * 64, n0, n0 + n1, S0 > 0, S1 > 0);
    };
    auto reduce = [&](auto vec, auto one_pass) __attribute__((always_inline)) {
        reduce_slots<DT, D, decltype(vec)::value, decltype(one_pass)::value>(R, sm.ml, sm_o, head0, G, W * 64, n0, n1, S0 > 0, S1 > 0);
    };
    constexpr std::integral_constant<int, 1> one;
    constexpr std::integral_constant<int, 2> two;
    constexpr std::integral_constant<int, 4> four;
    if (W < kFewSlots)
        G * D <= W * 64 ? few(one) : few(four);
    else if (G * D <= 256)
        reduce(one, std::true_type());
    else if (G * D <= 512)
        reduce(two, std::true_type());
    else
        reduce(four, std::false_type());
}

}  // namespace spd
