// Partial attention over one chunk of one (user, KV head): bf16, fp16 or fp32 K/V, head_dim D = 128 or 64, MFMA path.
//
// What it computes (paper section 4.2): for each of the G query heads that share this KV head,
//   A = softmax(s) V and lse = ln sum exp(s) over the chunk's tokens, s_i = scale * <q, k_i>,
// i.e. one owner's term of Theorem 1 restricted to a token range.  Chunks of one row are later
// combined with the n-way form of the same theorem (combine.hpp).
//
// Mapping onto a 64-lane wave (r = lane % 16, grp = lane / 16), 32 tokens per step (16 for 512-byte rows):
//   S^T = K . Q^T   two v_mfma_f32_16x16x32_{bf16,f16} chains (D/32 MFMAs each):
//                   the A operand is K as loaded (lane reads 16 B = 8 channels of token row r),
//                   the B operand is Q (head r, rows >= G are zero).  The result lands with
//                   head = r and tokens tb + grp*8 + e (e = 0..7) in each lane.
//   softmax         online (running max m, running sum l) per lane; the max is made uniform across the
//                   four lane groups of a head with two cross-lane exchanges per step.
//   O^T += V^T P^T  D/16 MFMA pairs (one per channel phase cc): the A operand V^T needs 8 tokens of one
//                   channel per lane; the lane loaded D/16 channels of 8 tokens (16 B each at D = 128, 8 B
//                   at D = 64: 16 lanes read a full row either way), so the operand is formed in registers
//                   with v_perm_b32 (no LDS).
//                   P is split into hi + lo parts of the element type, so the product keeps ~16 (bf16) or ~22
//                   (fp16) mantissa bits.  fp16 has a narrow exponent range: there P carries a factor 2^14 (the
//                   running sum l carries it too, so it cancels in A; lse subtracts it), which keeps
//                   probabilities down to 4e-9 of the row's largest out of the subnormal range.
//                   The B operand P^T is exactly the lane's own 8 probabilities.
// fp32 inputs take the same route with v_mfma_f32_16x16x4_f32 (one k-value per lane instead of eight): the lane's
// loads, the token each of its values belongs to and the layout of the results are the same as above, only the
// number of MFMAs per step differs (D/4 for S^T, D/2 for O^T at fp32, against D/16 and D/8 at 16 bits); P needs no
// split.
// fp32 with at most four query heads per KV head (kF32Quad; in this kernel with D = 128 only, in the whole-rows kernel at either
// D) takes v_mfma_f32_4x4x1_16b_f32 instead, sixteen independent
// 4x4 products per instruction at the same rate: the 16x16 tile spends 32 cycles on sixteen head columns of which G
// hold a head, 4096 cycles per 32 tokens at D = 128 (1.7 us in which no other wave of the SIMD has the pipe); the 4x4
// blocks need 1024.  With r = 4 * rq + i and NE tokens per lane group and step (8, or 4 with 512-byte rows), block (grp, rq) of
// S^T takes tokens tb + grp*NE + a*4 + i and the
// 16-byte piece rq of every 64 channel bytes (the four pieces are then summed over rq inside the 16-lane row with DPP
// adds), so a lane ends up with head i and tokens tb + grp*NE + e, exactly the P that block (grp, rq) of O^T needs for
// channels o_channel(4*rq + i, cc).  O^T stays split over grp (disjoint tokens) until the segment ends.
// fp32 rows of 512 bytes (D = 128) are HBM-bound once three things are so (8B shape, 16 users of 512-4096 tokens, 338 MB,
// us per fused step): the 4x4 blocks 73.9 -> 71.7; a lane's V loads cover 256 contiguous bytes per instruction instead
// of every other 16 (whose lines were asked for twice) -> 64.6; a wave's step is 16 tokens, 16 KB as at 16 bits, so that
// three waves per SIMD fit and the public owner's pieces start with the private ones -> 62.1 (5.5 TB/s).  Two 16-token
// steps in flight with two waves per SIMD: 64.4; the same order on 10.9 GB (1667 against 1702, before 1915).
// Every K/V byte is read once per KV head (all G heads share the tile).
// The four waves of a workgroup take interleaved 32-token steps and are combined through LDS; the result rows of a
// workgroup that crosses many rows wait in LDS too and are stored together (the result ring, below).
#pragma once
#include "common.hpp"

namespace spd {

// The element type's MFMA and conversions, by dtype code (SPD_BF16 / SPD_F16: an integer template argument keeps
// the kernel's name readable in profiler output).
template <int DT>
struct Elt;
template <>
struct Elt<SPD_BF16> {
    static constexpr int kBytes = 2;
    typedef __bf16 type;
    typedef __bf16 vec8 __attribute__((ext_vector_type(8)));
    static constexpr float kPShift = 0.f;  // log2 of the factor P carries into the second MFMA
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <>
struct Elt<SPD_F16> {
    static constexpr int kBytes = 2;
    typedef _Float16 type;
    typedef _Float16 vec8 __attribute__((ext_vector_type(8)));
    static constexpr float kPShift = 14.f;  // P <= 2^14 < 65504
    static __device__ __forceinline__ f32x4 mfma(vec8 a, vec8 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

template <>
struct Elt<SPD_F32> {
    static constexpr int kBytes = 4;
    static constexpr float kPShift = 0.f;
    static __device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

// fp32 with at most four query heads per KV head: the kernels' own dtype code for the 4x4 blocks (see above).
constexpr int kF32Quad = 3;
constexpr int kQuadHeads = 4;
template <>
struct Elt<kF32Quad> {
    static constexpr int kBytes = 4;
    static constexpr float kPShift = 0.f;
    static __device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
    }
};

// The same arithmetic in the streaming kernel's other forms (D = 128), by dtype codes of its own: 16-bit elements in steps of 16
// tokens ("half steps"), and kF32Quad with its rows read through buffer descriptors, as the half steps read theirs where they can
// (contiguous rows without an append).
// What half steps are for: a round of 16 KB per wave takes ~3.6 us while everything streams, a piece of 17 steps is five rounds to one
// wave and four to the other three, and nothing is in flight while a wave computes: rounds of half the size leave less of both at a
// piece's end.  Measured, us per fused step, 32-token steps / half steps: 16 users of 512-4096 + 1-512 tokens 33.2 / 32.6, with the
// append 34.1 / 33.2, in 16-token pages 33.8 / 32.7, both 34.4 / 32.8, as two parties 40.4 / 40.2; 12 such users 27.1 / 26.3, 24
// 46.9 / 46.0; 8 users of 4000-12000 49.8 / 48.7, 2 of 20000-40000 48.2 / 46.8; workload 2 itself the same within its noise (31.0 /
// 31.0, with the append 32.0 / 31.7, as two parties 37.8 / 37.4).  They take 10 % more vector instructions per token (workload 2:
// 3.50 M against 3.17 M).
// In buffer descriptors a lane's offset and a scalar per row are all the addressing there is: fp32, 16 such users, 60.9 / 60.0 (workload
// 2's lengths 55.4 / 55.0; vector instructions 4.25 M / 3.73 M).
// An append reads its last row elsewhere, and one instance serves a launch: it keeps plain addresses for both owners.  Contiguous rows
// then gain by how the rounds divide (14 users 30.8 / 31.1, 16 34.1 / 33.2, 18 37.6 / 37.4, 20 40.4 / 39.3, 24 47.2 / 47.7, 32 60.5 / 60.5).
constexpr int kFormStep = 3;  // from a dtype's code to its other form's
constexpr int kBf16Half = SPD_BF16 + kFormStep, kF16Half = SPD_F16 + kFormStep, kF32QuadRange = kF32Quad + kFormStep;
constexpr int form_of(int dt) { return dt >= kBf16Half ? 1 : 0; }
template <>
struct Elt<kBf16Half> : Elt<SPD_BF16> {};
template <>
struct Elt<kF16Half> : Elt<SPD_F16> {};
template <>
struct Elt<kF32QuadRange> : Elt<kF32Quad> {};
constexpr bool half_steps(int dt) { return dt == kBf16Half || dt == kF16Half; }
constexpr bool quad_blocks(int dt) { return dt == kF32Quad || dt == kF32QuadRange; }
constexpr bool by_descriptor(int dt, bool paged, bool append) { return (half_steps(dt) || dt == kF32QuadRange) && !paged && !append; }

// Sum over the four lanes of a 16-lane row that differ in bits 2 and 3 (rq), in all of them: two rotations of the row.  By eight first:
// each lane then adds the same two pairs, so all four get the same bits.  (By four first they add different pairs: scores, and with them
// the running maxima, differ in the last bit between the lanes that hold a head's channels, and a wave's state, handed over with one
// lane's maximum, is off by what that is worth: 4e-5 at scores of 500, 2 % more error at ordinary ones.)
__device__ __forceinline__ float row_quad_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));  // row_ror:8
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, true));  // row_ror:4
    return v;
}

// Sums an accumulator that is split over the four lane groups, each group keeping a quarter of the channel phases: on
// return acc[0 .. CP/4) of lane group grp holds the totals of phases (grp >> 1) * CP/2 + (grp & 1) * CP/4 + k.
// (A swap of half the lanes between two phases' registers brings each phase's two halves into the same lanes.)
template <int CP>
__device__ __forceinline__ void reduce_scatter_groups(f32x4 (&acc)[CP])
{
#pragma unroll
    for (int k = 0; k < CP / 2; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[k][v]), __float_as_uint(acc[k + CP / 2][v]), false, false);
            acc[k][v] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
#pragma unroll
    for (int k = 0; k < CP / 4; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[k][v]), __float_as_uint(acc[k + CP / 4][v]), false, false);
            acc[k][v] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
}

// One step's loads of a lane, for rows of RB bytes (D channels of 2 or 4 bytes): RB/64 16-byte pieces of each of its
// two K rows, and RB/16 bytes (D/16 channels) of each of its eight V rows.
// A lane's share of one V row (RB/16 bytes), kept in the registers its loads deliver it in.
template <int RB>
struct VRow;
template <>
struct VRow<128> {
    u32x2 w;
    __device__ __forceinline__ void load(const char *p) { w = stream_load<u32x2>(p); }
    __device__ __forceinline__ unsigned dword(int i) const { return w[i]; }
};
template <>
struct VRow<256> {
    u32x4 w;
    __device__ __forceinline__ void load(const char *p) { w = stream_load16(p); }
    __device__ __forceinline__ void load(row_rsrc b, unsigned at) { w = stream_load16(b, at); }
    __device__ __forceinline__ unsigned dword(int i) const { return w[i]; }
};
template <>
struct VRow<512> {
    u32x4 w0, w1;  // 16 bytes of each half of the row, so that an instruction's sixteen lanes cover 256 contiguous bytes
    __device__ __forceinline__ void load(const char *p)
    {
        w0 = stream_load16(p);
        w1 = stream_load16(p + 256);
    }
    __device__ __forceinline__ void load(row_rsrc b, unsigned at)
    {
        w0 = stream_load16(b, at);
        w1 = stream_load16(b, at + 256);
    }
    __device__ __forceinline__ unsigned dword(int i) const { return i < 4 ? w0[i] : w1[i - 4]; }  // i is a constant
};

// Lane r's first byte of a V row is r * v_lane_bytes(RB).
__host__ __device__ constexpr int v_lane_bytes(int RB) { return RB == 512 ? 16 : RB / 16; }

// The channel that row `row` (0..15) of the O^T tile's phase cc (0..CP-1) holds: lane r = row loaded it as value cc of its
// share of a V row.
template <int RB, int CP>
__device__ __forceinline__ constexpr int o_channel(int row, int cc)
{
    return RB == 512 ? (cc >> 2) * 64 + row * 4 + (cc & 3) : row * CP + cc;
}

// 16-token S tiles per step of a wave: two, or one where rows are 512 bytes (fp32 with D = 128), so that a step is 16 KB
// at either row size; half that in half steps.
__host__ __device__ constexpr int step_tiles(int RB, bool half = false) { return RB == 512 || half ? 1 : 2; }
__host__ __device__ constexpr int step_tokens(int RB) { return 16 * step_tiles(RB); }

template <int RB, int NA>
struct TileRegs {
    u32x4 k[NA][RB / 64];  // [S tile a][piece kk]: token row kt of tile a, bytes kk*64 + kc*16 .. +16 (see LaneConst)
    VRow<RB> v[4 * NA];    // [e]: token tb + grp*NE + e, RB/16 bytes from r*v_lane_bytes on
};

struct LaneConst {
    int r, grp;
    int kt, kc;  // the lane's K rows: tokens tb + kt*NE + a*4 + (r & 3) (NE = 4 * step_tiles), 16-byte piece kc (r / 4 and grp; kF32Quad: grp and r / 4)
    const char *k_base;  // contiguous: user's K + head offset; paged: pool + head offset
    const char *v_base;
    const int32_t *bt_row;
    int page_shift, page_mask;  // paged: token t lies in the row's page t >> page_shift at place t & page_mask
    int64_t token_stride, block_stride;
    const char *k_new_row;  // KV append: this (user, KV head)'s new K / V row if the segment ends its row, else nullptr
    const char *v_new_row;
};

// The pages that hold the two 16-token halves of the 32-token step at tb (the same page twice if pages hold 32 tokens
// or more).  The ids are wave-uniform and come through the scalar cache.  Clamping keeps the lookups inside the
// user's pages; rows past the chunk re-read its last token, which lies in the page the clamped lookup names (an
// 8-token group never straddles a page).
struct PagePair {
    int p0, p1;
};

__device__ __forceinline__ PagePair load_pages(const LaneConst &L, int tb, int t_last)
{
    const int tbu = uniform(tb);
    PagePair P;
    P.p0 = scalar_load_i32(L.bt_row, min(tbu, t_last) >> L.page_shift);
    P.p1 = scalar_load_i32(L.bt_row, min(tbu + 16, t_last) >> L.page_shift);
    return P;
}

// Issues the loads of the step at tb, NA 16-token tiles.  Paged: P holds that step's page ids on entry and the following step's
// (tb + step) on return: the lookup is issued behind the data loads, one whole step before it is needed, so that no
// wave ever waits for a block-table entry before it can ask for data.
// RANGE: through buffer descriptors whose range ends with the segment (rows past it are zeros and cost no traffic), for rows that lie
// end to end.  (Their stride is read all the same: with constant offsets 16 users of 512-4096 + 1-512 tokens take the same time, but 16
// of 1000-3000 + 1000-3000 tokens 92.3 us instead of 88.4, 4 such 32.5 instead of 31.4.)
template <int RB, int NA, bool PAGED, bool APPEND, bool RANGE = false>
__device__ __forceinline__ void load_tile(TileRegs<RB, NA> &T, const LaneConst &L, int tb, int t_last, PagePair &P, int step)
{
    constexpr int NE = 4 * NA;
    if constexpr (RANGE) {
        static_assert(!PAGED && !APPEND);
        // (the whole offset is the lane's, see row_buffer: 3 registers more than with scalar parts for the tokens, fp32 6, and the same time)
        const unsigned stride = (unsigned)L.token_stride;
        const unsigned k_lane = (L.kt * NE + (L.r & 3)) * stride + L.kc * 16, v_lane = L.grp * NE * stride + L.r * v_lane_bytes(RB);
        const row_rsrc kb = row_buffer(L.k_base, tb, t_last, L.token_stride, RB), vb = row_buffer(L.v_base, tb, t_last, L.token_stride, RB);
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int kk = 0; kk < RB / 64; ++kk)
                T.k[a][kk] = stream_load16(kb, k_lane + a * 4 * stride + kk * 64);
#pragma unroll
        for (int e = 0; e < NE; ++e)
            T.v[e].load(vb, v_lane + e * stride);
        __builtin_amdgcn_sched_barrier(0);
        return;
    }
    const int gk = tb + L.kt * NE;       // first token of the NE-token group this lane's K rows fall in
    const int gv = tb + L.grp * NE;      // first token of the group this lane's V rows fall in
    const char *kp = L.k_base, *vp = L.v_base;
    if (PAGED) {
        kp += (int64_t)((gk - tb) >= 16 ? P.p1 : P.p0) * L.block_stride;
        vp += (int64_t)((gv - tb) >= 16 ? P.p1 : P.p0) * L.block_stride;
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int t = min(gk + a * 4 + (L.r & 3), t_last);  // rows past the chunk re-read its last token (masked later)
        const char *p = kp + (int64_t)(PAGED ? (t & L.page_mask) : t) * L.token_stride + L.kc * 16;
        if (APPEND && L.k_new_row && t == t_last)  // the appended token is read from the caller's buffer, not the cache
            p = L.k_new_row + L.kc * 16;
#pragma unroll
        for (int kk = 0; kk < RB / 64; ++kk)
            T.k[a][kk] = stream_load16(p + kk * 64);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int t = min(gv + e, t_last);
        const char *p = vp + (int64_t)(PAGED ? (t & L.page_mask) : t) * L.token_stride + L.r * v_lane_bytes(RB);
        if (APPEND && L.v_new_row && t == t_last)
            p = L.v_new_row + L.r * v_lane_bytes(RB);
        T.v[e].load(p);
    }
    if (PAGED)
        P = load_pages(L, tb + step, t_last);
    // all loads of the step are issued before anything that follows: without this the compiler sinks the V loads
    // below the K wait to shorten live ranges, which serialises two memory round trips per step
    __builtin_amdgcn_sched_barrier(0);
}

// qB: Q as the B operand, loaded like a K row (head r instead of token r): bytes kk*64 + kc*16 .. +16 of the row.
template <int DT, int D, int NA>
__device__ __forceinline__ void compute_tile(const TileRegs<D * Elt<DT>::kBytes, NA> &T,
                                             const u32x4 (&qB)[D * Elt<DT>::kBytes / 64], int tb, int grp, int t_end,
                                             float c, float &m, float &l, f32x4 (&acc)[D / 16])
{
    constexpr int RB = D * Elt<DT>::kBytes;
    constexpr int NE = 4 * NA;
    f32x4 s[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a)
        s[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (Elt<DT>::kBytes == 4) {
#pragma unroll
        for (int kk = 0; kk < RB / 64; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e)  // four channels per piece, one MFMA (k = 4: the lane groups; k = 1 in 4x4 blocks) each
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    s[a] = Elt<DT>::mfma(__uint_as_float(T.k[a][kk][e]), __uint_as_float(qB[kk][e]), s[a]);
    } else {
        typedef typename Elt<DT>::vec8 vec8;
#pragma unroll
        for (int kk = 0; kk < RB / 64; ++kk)
#pragma unroll
            for (int a = 0; a < NA; ++a)
                s[a] = Elt<DT>::mfma(__builtin_bit_cast(vec8, T.k[a][kk]), __builtin_bit_cast(vec8, qB[kk]), s[a]);
    }
    if constexpr (quad_blocks(DT)) {  // the four 16-byte pieces of every 64 channel bytes
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s[a][e] = row_quad_sum(s[a][e]);
    }
    // scores in log2 units; tokens past the chunk end get -inf
    const int t0 = tb + grp * NE;
    float x[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e)
        x[e] = (t0 + e < t_end) ? s[e / 4][e % 4] * c : -INFINITY;
    float mt = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    if constexpr (NE == 8)
        mt = fmaxf(mt, fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    mt = wave_xor_max<16>(mt);
    mt = wave_xor_max<32>(mt);
    const float m_new = fmaxf(m, mt);  // finite: every step holds at least one token of the chunk
    const float alpha = fast_exp2(m - m_new);
    const float m_p = m_new - Elt<DT>::kPShift;  // p (and with it l and acc) carries the factor 2^kPShift
    float p[NE], ps = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        p[e] = fast_exp2(x[e] - m_p);
        ps += p[e];
    }
    l = l * alpha + ps;
    m = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {  // wave-uniform: rescale only when some max moved
#pragma unroll
        for (int cc = 0; cc < D / 16; ++cc)
            acc[cc] *= alpha;
    }
    if constexpr (quad_blocks(DT)) {
        // a block per lane-group token and four of the lane's channels; the phases are independent chains
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int cc = 0; cc < D / 16; ++cc)
                acc[cc] = Elt<DT>::mfma(__uint_as_float(T.v[e].dword(cc)), p[e], acc[cc]);
    } else if constexpr (DT == SPD_F32) {
        // channel phase cc: the lane's dword cc of each of its tokens; the MFMA's four k-values are the four
        // lane groups' tokens grp*NE + e, and the B operand is the lane's own probability of that token
#pragma unroll
        for (int cc = 0; cc < D / 16; ++cc)
#pragma unroll
            for (int e = 0; e < NE; ++e)
                acc[cc] = Elt<DT>::mfma(__uint_as_float(T.v[e].dword(cc)), p[e], acc[cc]);
    } else if constexpr (NA == 1) {
        // four tokens to a lane: the high and the low parts of their probabilities fill one operand, the V values the other twice
        typedef typename Elt<DT>::vec8 vec8;
        typedef typename Elt<DT>::type E;
        vec8 pp;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pp[e] = (E)p[e];
            pp[e + 4] = (E)(p[e] - (float)pp[e]);
        }
#pragma unroll
        for (int cc = 0; cc < D / 16; ++cc) {
            const unsigned sel = (cc & 1) ? 0x07060302u : 0x05040100u;
            u32x4 vt;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                vt[j] = vt[j + 2] = __builtin_amdgcn_perm(T.v[2 * j + 1].dword(cc >> 1), T.v[2 * j].dword(cc >> 1), sel);
            acc[cc] = Elt<DT>::mfma(__builtin_bit_cast(vec8, vt), pp, acc[cc]);
        }
    } else {
        typedef typename Elt<DT>::vec8 vec8;
        typedef typename Elt<DT>::type E;
        vec8 ph, pl;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            ph[e] = (E)p[e];
            pl[e] = (E)(p[e] - (float)ph[e]);
        }
#pragma unroll
        for (int cc = 0; cc < D / 16; ++cc) {
            const int w = cc >> 1;
            const unsigned sel = (cc & 1) ? 0x07060302u : 0x05040100u;  // odd channel: high halves, even: low halves
            u32x4 vt;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                vt[j] = __builtin_amdgcn_perm(T.v[2 * j + 1].dword(w), T.v[2 * j].dword(w), sel);  // (token 2j, token 2j+1) of channel cc
            const vec8 va = __builtin_bit_cast(vec8, vt);
            acc[cc] = Elt<DT>::mfma(va, ph, acc[cc]);
            acc[cc] = Elt<DT>::mfma(va, pl, acc[cc]);
        }
    }
}

// LDS row stride (floats) of one head's D channels: the four extra floats spread the heads over the banks
__host__ __device__ constexpr int o_stride(int D) { return D + 4; }

// LDS bytes of the result staging tiles of a workgroup of `waves` waves, and whether the head-per-wave mapping can have
// them (kernel and launch use the same rule; 64 KB is what a workgroup may ask for without special attributes).
__host__ __device__ constexpr size_t staging_bytes(int D, int waves, int G)
{
    return sizeof(float) * (size_t)waves * G * o_stride(D);
}
__host__ __device__ constexpr bool staging_fits(int D, int waves, int G) { return staging_bytes(D, waves, G) <= 64 * 1024; }

// The result ring.  A piece that crosses rows produces a result row ([G][D] values and G log-sum-exps, final or a chunk
// partial) at every segment end.  Written where they arise, those rows reach HBM as single lines scattered over the
// read stream, and each costs the memory system far more than its bytes: a plain streaming read of 2.8 GB at 768
// workgroups takes 414 us, 444 us with 8 MB of such rows written along the way, and 418 us with the same rows written
// when a workgroup is done (measured on this GPU; workload 4 writes 8 MB of them in 443 us).  So a head-major
// workgroup keeps its rows in LDS, up to `ring_rows` of them, and stores them together when the ring is full or the
// piece ends.  A row of the ring: G * D values, then G log-sum-exps, padded to a multiple of four floats.
constexpr int kRingMaxRows = 32;
__host__ __device__ constexpr int ring_row_floats(int D, int G) { return G * D + ((G + 3) & ~3); }
// LDS bytes a head-major workgroup may use for staging and ring together: a CU's 160 KB are shared by the three
// workgroups that the one-step kernel's registers allow, or by two (the two-step kernel, or a launch of no more than
// two workgroups per CU), and a workgroup may ask for 64 KB in all.
__host__ __device__ constexpr size_t ring_lds_budget(bool two_per_cu) { return (two_per_cu ? 60 : 40) * 1024; }
__host__ __device__ constexpr int ring_rows_that_fit(int D, int G, bool two_per_cu)
{
    const size_t staging = sizeof(float) * (size_t)kWaves * G * o_stride(D);
    const size_t row = sizeof(float) * (size_t)ring_row_floats(D, G);
    const size_t n = staging >= ring_lds_budget(two_per_cu) ? 0 : (ring_lds_budget(two_per_cu) - staging) / row;
    return n < 2 ? 0 : n > (size_t)kRingMaxRows ? kRingMaxRows : (int)n;  // a ring of one row holds nothing back
}

// The same for the head-per-wave mapping, where every wave owns a row per segment: a ring per wave, its rows in the
// layout of the wave's staging tile ([G][o_stride]), then G log-sum-exps (padded to four floats) and the two pointers
// the row goes to.
__host__ __device__ constexpr int hpw_ring_row_floats(int D, int G) { return G * o_stride(D) + ((G + 3) & ~3) + 4; }
__host__ __device__ constexpr int hpw_ring_rows_that_fit(int D, int G, int waves)
{
    const size_t staging = sizeof(float) * (size_t)waves * G * o_stride(D);
    const size_t row = sizeof(float) * (size_t)hpw_ring_row_floats(D, G) * waves;
    const size_t n = staging >= ring_lds_budget(true) ? 0 : (ring_lds_budget(true) - staging) / row;
    return n < 2 ? 0 : n > (size_t)kRingMaxRows ? kRingMaxRows : (int)n;
}

// Waves per SIMD the kernel is compiled for: a step's loads take 64 registers per lane (32 with rows of 128 bytes), twice
// that with PREFETCH.
__host__ __device__ constexpr int mfma_waves_per_simd(int RB, bool prefetch, bool hpw)
{
    return RB >= 256 ? (prefetch ? 2 : 3) : (hpw ? 2 : 3);
}

// One workgroup per piece (see DevItem); q: [U][Hq][D] of the element type DT (SPD_BF16, SPD_F16 or SPD_F32).  A
// segment that is its row's only one writes out/lse directly; otherwise it writes part_o[slot][G][D] /
// part_lse[slot][G], which combine_chunks_kernel then reduces.
//
// (Register counts below are those of 256-byte rows: 16-bit elements with D = 128.  Rows of 128 bytes need about half
// and always run with PREFETCH; fp32 rows of 512 bytes need ~160 with one 16-token step in flight and never run with it.)
// PREFETCH = true keeps two 32-token steps of loads in flight per wave (~245 VGPRs, two waves per SIMD): for launches
// that run several rounds of workgroups, and for small ones that fit two per CU anyway (half as many dependent round
// trips per wave).  PREFETCH = false holds one step (~160 VGPRs, three waves per SIMD; half steps 132-137): as fast when the private
// owner's pieces are one resident round, and it leaves room on every CU for the other owner's pieces.
//
// HPW ("head per wave") is the mapping for contiguous token-major storage, where the KV heads of a token are adjacent
// in memory ([token][head][d]).  A piece is then a token range of a *user* for a group of two to eight KV heads (the
// host picks the group size by the size of the launch), the workgroup has one wave per KV head of the group, and all waves walk the same tokens:
// together they read whole, consecutive DRAM pages, where one workgroup per head would touch every page eight times
// at different moments (a barrier per step keeps the waves together).  Each wave owns its head's result, so there is no cross-wave combine; the wave stores its
// result through an LDS tile of its own.  Without HPW (head-major storage: one contiguous stream per head) a piece is
// a token range of one (user, KV head) row and its four waves take interleaved steps.
//
// APPEND = true adds the KV append (the address substitution costs ~1 % when nothing is appended, hence a flag).
// CHANNELS = -D is the dtype's other form (see form_of): so the first argument stays the dtype, and a profile's names of the other
// instances stay what they are in stored ones.  (A body shared by two kernel templates costs registers: workload 5 +3 %.)
template <int DTYPE, int CHANNELS, bool PAGED, bool PREFETCH, bool HPW, bool APPEND>
__global__ __launch_bounds__(HPW ? 512 : kThreads,
                             mfma_waves_per_simd((CHANNELS < 0 ? -CHANNELS : CHANNELS) * Elt<DTYPE>::kBytes, PREFETCH, HPW)) void partial_mfma_kernel(
    u32x8 head_a, u32x4 head_b, u32x2 head_c, PartialArgs)  // see PartialHead
{
    const PartialHead H = head_of<PartialHead>(head_a, head_b, head_c);
    const int n0 = H.n0, Hq = H.Hq, G = H.G, ring_rows = H.ring_rows;
    const float scale_log2e = H.scale_log2e;
    const Address q = (Address)H.q;
    constexpr int D = CHANNELS < 0 ? -CHANNELS : CHANNELS;
    constexpr int DT = CHANNELS < 0 ? DTYPE + kFormStep : DTYPE;
    const bool second = (int)blockIdx.x >= n0;  // workgroup-uniform: which owner this workgroup serves
    const DevItem *__restrict__ items = second ? H.items[1] : H.items[0];
    const int grow = second ? H.grow[1] : H.grow[0];
    DevItem it = grown(scalar_load_item(items, second ? (int)blockIdx.x - n0 : (int)blockIdx.x), grow);
    // The owner's arguments come beside the item, at an address of their own (a field chosen from either owner's is two addresses and a
    // selection each), and there is one wait for all that the first tile needs: as the compiler placed them, up to six round trips
    // stood in front of it.  With the preloaded head, us per call before / after: 16 users of 512-4096 + 1-512 tokens fused 32.46 / 31.98,
    // token-major as two parties with the append 43.43 / 42.28; launches of 0.2 ms and more are the same.
    const auto own = (const OwnerArgs __attribute__((address_space(4))) *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
                                                                          kPartialArgsAt + (second ? (int)sizeof(OwnerArgs) : 0));
    const KvAddr kv = {own->kv.block_table, own->kv.max_blocks, own->kv.page_shift, own->kv.block_stride, own->kv.token_stride, own->kv.head_stride};
    const uintptr_t k_pool = reinterpret_cast<uintptr_t>(own->k_pool), v_pool = reinterpret_cast<uintptr_t>(own->v_pool);  // 0 unless paged
    const char *const *k_ptrs = own->k_ptrs, *const *v_ptrs = own->v_ptrs;  // null unless the view brought device pointer tables
    const char *k_new = own->k_new, *v_new = own->v_new;
    float *__restrict__ out = own->out, *__restrict__ lse = own->lse;
    float *__restrict__ part_o = own->part_o, *__restrict__ part_lse = own->part_lse;
    asm volatile("" ::"s"(it.k_base), "s"(it.v_base), "s"(it.user), "s"(it.rot), "s"(k_ptrs), "s"(v_ptrs), "s"(kv.token_stride), "s"(out));
    if constexpr (PAGED)
        asm volatile("" ::"s"(k_pool), "s"(v_pool), "s"(kv.block_table), "s"(kv.max_blocks), "s"(kv.page_shift), "s"(kv.block_stride));
    __shared__ float2 sm_ml[kWaves][16];  // running max and sum of every wave
    __shared__ float *ring_dst_o[kRingMaxRows], *ring_dst_l[kRingMaxRows];  // where the ring's rows go
    extern __shared__ __align__(16) float sm_o[];  // [waves][G * kOStride], sized by the launch: only G heads are staged; then the ring
    constexpr int kOStride = o_stride(D);
    constexpr int CP = D / 16;  // channel phases of the O^T tile; which channel a phase of a row holds: o_channel
    constexpr int kRowBytes = D * Elt<DT>::kBytes;
    constexpr int RB = kRowBytes;
    constexpr bool kQuad = quad_blocks(DT);
    constexpr bool kHalf = half_steps(DT), kRange = by_descriptor(DT, PAGED, APPEND);
    constexpr int NA = step_tiles(RB, kHalf);  // 16-token tiles of a wave's step
    const int o_wave_stride = G * kOStride;
    // head-per-wave results go through a wave-private tile if the launch gave the room
    const bool staged = HPW && staging_fits(D, (int)(blockDim.x >> 6), G);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    constexpr int kTile = 16 * NA;  // tokens per step of a wave
    constexpr int kStep = HPW ? kTile : kTile * kWaves;

    // Everything a segment needs before its first MFMA: addresses, the KV append copy, Q, and the loads of the wave's
    // first 32-token step.  Issued for the *next* segment before the current one's epilogue, so that the barriers
    // and the result stores of the epilogue overlap the memory round trip instead of preceding it.
    auto begin_segment = [&](const DevItem &it, LaneConst &L, u32x4 (&qB)[RB / 64], int &tb, TileRegs<RB, NA> &T0, PagePair &P) {
        L.r = lane & 15;
        L.grp = lane >> 4;
        L.kt = kQuad ? L.grp : L.r >> 2;
        L.kc = kQuad ? L.r >> 2 : L.grp;
        L.token_stride = kv.token_stride;
        L.block_stride = kv.block_stride;
        L.page_shift = kv.page_shift;
        L.page_mask = (1 << kv.page_shift) - 1;
        const int kv_head = HPW ? it.kv_head + uniform(wave) : it.kv_head;  // head per wave: the group's first head + wave
        L.k_base = it.k_base + k_pool + (PAGED ? 0 : user_base(k_ptrs, it.user)) + (HPW ? (int64_t)kv_head * kv.head_stride : 0);
        L.v_base = it.v_base + v_pool + (PAGED ? 0 : user_base(v_ptrs, it.user)) + (HPW ? (int64_t)kv_head * kv.head_stride : 0);
        L.bt_row = PAGED ? kv.block_table + (int64_t)it.user * kv.max_blocks : nullptr;
        const int t_last = it.t_end - 1;
        L.k_new_row = L.v_new_row = nullptr;
        if (APPEND && k_new && (it.rot & kEndsRow)) {
            // KV append: this segment holds the row's last token, which is the new one.  Wave 0 copies its K and V
            // rows into the cache (16 bytes per lane, K in the first lanes, V in the next); every reader of that token
            // takes it from the caller's buffer instead, so nothing waits for the copy.
            constexpr int kRowLanes = kRowBytes / 16;
            const int64_t row = ((int64_t)it.user * (Hq / G) + kv_head) * kRowBytes;
            L.k_new_row = k_new + row;
            L.v_new_row = v_new + row;
            if ((HPW || wave == 0) && lane < 2 * kRowLanes) {
                int64_t off = (int64_t)(PAGED ? (t_last & L.page_mask) : t_last) * kv.token_stride + (lane % kRowLanes) * 16;
                if (PAGED)
                    off += (int64_t)scalar_load_i32(L.bt_row, t_last >> L.page_shift) * kv.block_stride;
                if (lane < kRowLanes)
                    copy16(const_cast<char *>(L.k_base) + off, L.k_new_row + lane * 16);
                else
                    copy16(const_cast<char *>(L.v_base) + off, L.v_new_row + (lane - kRowLanes) * 16);
            }
        }
        // Q as the B operand: head r (4x4 blocks: r & 3; zero beyond G), read like a K row: bytes kk*64 + kc*16 .. +16
        const int head = kQuad ? L.r & (kQuadHeads - 1) : L.r;
        const Address qrow = q + ((int64_t)it.user * Hq + (int64_t)kv_head * G + head) * kRowBytes + L.kc * 16;
#pragma unroll
        for (int kk = 0; kk < RB / 64; ++kk) {
            qB[kk] = u32x4{0u, 0u, 0u, 0u};
            if (head < G)
                qB[kk] = *(const u32x4 __attribute__((address_space(1))) *)(qrow + kk * 64);
        }
        // head-major: the four waves take interleaved steps (rot counts 32-token ones); token-major: every wave takes every step
        tb = HPW ? it.t_begin : it.t_begin + ((uniform(wave) - (kHalf ? 2 * it.rot : it.rot)) & (kWaves - 1)) * kTile;
        if (PAGED)
            P = load_pages(L, tb, t_last);
        if (PREFETCH && tb < it.t_end)
            load_tile<RB, NA, PAGED, APPEND, kRange>(T0, L, tb, t_last, P, kStep);
    };

    if (it.n_chunks == 0) {  // a row without tokens (head-per-wave: a user without tokens) is a piece of its own
        if (HPW) {
            const int64_t head0 = (int64_t)it.user * Hq + (int64_t)(it.kv_head + wave) * G;
            for (int idx = lane; idx < G * D; idx += 64)
                out[head0 * D + idx] = 0.f;
            if (lane < G)
                lse[head0 + lane] = -INFINITY;
        } else {
            write_empty_row<D>(it, G, Hq, out, lse);
        }
        return;
    }
    LaneConst L;
    u32x4 qB[RB / 64];
    int tb;
    TileRegs<RB, NA> T0;
    PagePair P = {0, 0};
    int n_ring = 0;  // rows held in the result ring (head-major mapping only)
    begin_segment(it, L, qB, tb, T0, P);
    for (;;) {
        // the piece's next segment is fetched (scalar cache) long before it is looked at: with tens of MB of loads in
        // flight a dependent round trip costs microseconds, so none may sit between two segments.  (Its growth is applied there too:
        // here it would be a wait in front of the segment's first tile, and hold what the owner's arguments need: the instances for pages
        // with the append, which spill 20 scalar registers, spilled 39 with it, us per call 14.54 / 14.00, 32.74 / 31.55.)
        DevItem nx;
        if (it.next >= 0)
            nx = scalar_load_item(items, it.next);
        const int t_last = it.t_end - 1;

        float m = -INFINITY, l = 0.f;
        f32x4 acc[CP];
#pragma unroll
        for (int cc = 0; cc < CP; ++cc)
            acc[cc] = f32x4{0.f, 0.f, 0.f, 0.f};

        if (!PREFETCH) {
            for (; tb < it.t_end; tb += kStep) {
                TileRegs<RB, NA> T;
                load_tile<RB, NA, PAGED, APPEND, kRange>(T, L, tb, t_last, P, kStep);
                compute_tile<DT, D>(T, qB, tb, L.grp, it.t_end, scale_log2e, m, l, acc);
            }
        } else if (tb < it.t_end) {  // T0 already holds (the loads of) step tb
            {
                TileRegs<RB, NA> T1;
                for (;;) {
                    const int tb1 = tb + kStep;
                    const bool more1 = tb1 < it.t_end;
                    // head per wave: the waves stay in step (they all run the same trip counts), so that together they
                    // ask for whole consecutive token rows at about the same time
                    if (HPW)
                        __builtin_amdgcn_s_barrier();
                    if (more1)
                        load_tile<RB, NA, PAGED, APPEND>(T1, L, tb1, t_last, P, kStep);
                    compute_tile<DT, D>(T0, qB, tb, L.grp, it.t_end, scale_log2e, m, l, acc);
                    if (!more1)
                        break;
                    const int tb2 = tb1 + kStep;
                    const bool more2 = tb2 < it.t_end;
                    if (HPW)
                        __builtin_amdgcn_s_barrier();
                    if (more2)
                        load_tile<RB, NA, PAGED, APPEND>(T0, L, tb2, t_last, P, kStep);
                    compute_tile<DT, D>(T1, qB, tb1, L.grp, it.t_end, scale_log2e, m, l, acc);
                    if (!more2)
                        break;
                    tb = tb2;
                }
            }
        }

        // (half steps and 512-byte rows: what only the epilogue needs of the lane and thread index is computed there, not held across
        // the streaming loop, which opaque copies of them see to)
        int late_lane = lane;
        if constexpr (kHalf)
            asm("" : "+v"(late_lane));
        const int grp = late_lane >> 4, r = late_lane & 15;
        // the two-per-CU kernel has the registers to let the next segment's loads fly during the epilogue below
        if (PREFETCH && it.next >= 0) {
            nx = grown(nx, grow);
            begin_segment(nx, L, qB, tb, T0, P);
        }

        // ---- combine the lane groups (sum of l) ... ----
        l = wave_xor_sum<16>(l);
        l = wave_xor_sum<32>(l);
        const bool direct = it.n_chunks == 1;
        if (HPW) {
            // ... and that is all: the wave owns head `wave` of this token range.  Lane (r < G, grp) holds channels
            // (4*grp + v)*CP + cc of query head r: CP consecutive floats per v.
            const int kvh = it.kv_head + uniform(wave);
            const int64_t head0 = (int64_t)it.user * Hq + (int64_t)kvh * G;
            const int64_t slot = (int64_t)it.slot + (int64_t)uniform(wave) * it.n_chunks;  // it.slot: the group's first head
            const float inv = fast_rcp(l);  // l > 0: the segment holds at least one token
            float *res = direct ? out + head0 * D : part_o + slot * G * D;  // [G][D], contiguous
            float *res_l = direct ? lse + head0 : part_lse + slot * G;
            // the row waits in the wave's ring - unless the piece ends here with an empty ring, or there is no ring
            const bool last = it.next < 0;
            const bool to_ring = staged && ring_rows > 0 && !(last && n_ring == 0);
            const int hrow = hpw_ring_row_floats(D, G);
            float *const ring_w = sm_o + (int)(blockDim.x >> 6) * o_wave_stride + wave * ring_rows * hrow;
            if (staged) {
                // Through a wave-private LDS tile, so that the wave stores whole rows with consecutive lanes (storing
                // straight from the accumulator layout puts 16 bytes per lane into 16 different cache lines per
                // instruction; measured 2-3 % of the kernel on long token-major workloads).
                float *stage = to_ring ? ring_w + n_ring * hrow : sm_o + wave * o_wave_stride;
                if (r < G) {
                    float *dst = stage + r * kOStride + grp * 4 * CP;
#pragma unroll
                    for (int cc = 0; cc < CP; ++cc)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            dst[v * CP + cc] = acc[cc][v] * inv;  // channel (4*grp + v)*CP + cc
                }
                if (to_ring) {
                    if (r < G && grp == 0)
                        stage[o_wave_stride + r] = (m + fast_log2(l) - Elt<DT>::kPShift) * kLn2;  // m is in log2 units
                    if (lane == 0) {
                        float **dst = reinterpret_cast<float **>(stage + o_wave_stride + ((G + 3) & ~3));
                        dst[0] = res;
                        dst[1] = res_l;
                    }
                    ++n_ring;
                }
                __builtin_amdgcn_wave_barrier();  // same wave: LDS executes its writes before its reads
                if (!to_ring) {
                    for (int i = lane * 4; i < G * D; i += 256) {
                        const f32x4 w = *reinterpret_cast<const f32x4 *>(stage + (i / D) * kOStride + (i % D));
                        *reinterpret_cast<f32x4 *>(res + i) = w;
                    }
                } else if (last || n_ring == ring_rows) {
                    typedef __attribute__((address_space(1))) float *global_f32;
                    for (int k = 0; k < n_ring; ++k) {
                        const float *row = ring_w + k * hrow;
                        float *const *dst = reinterpret_cast<float *const *>(row + o_wave_stride + ((G + 3) & ~3));
                        const global_f32 o = (global_f32)dst[0];
                        for (int i = lane * 4; i < G * D; i += 256) {
                            const f32x4 w = *reinterpret_cast<const f32x4 *>(row + (i / D) * kOStride + (i % D));
                            *reinterpret_cast<__attribute__((address_space(1))) f32x4 *>(o + i) = w;
                        }
                        if (lane < G)
                            ((global_f32)dst[1])[lane] = row[o_wave_stride + lane];
                    }
                    n_ring = 0;
                }
                __builtin_amdgcn_wave_barrier();
            }
            if (r < G) {
                if (!staged) {
                    float *dst = res + r * D + grp * 4 * CP;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int c4 = 0; c4 < CP; c4 += 4) {
                            const f32x4 w = {acc[c4][v] * inv, acc[c4 + 1][v] * inv, acc[c4 + 2][v] * inv, acc[c4 + 3][v] * inv};
                            *reinterpret_cast<f32x4 *>(dst + v * CP + c4) = w;
                        }
                }
                if (grp == 0 && !to_ring)
                    res_l[r] = (m + fast_log2(l) - Elt<DT>::kPShift) * kLn2;  // m is in log2 units
            }
            if (last)
                return;
            if (!PREFETCH) {
                nx = grown(nx, grow);
                begin_segment(nx, L, qB, tb, T0, P);
            }
            it = nx;
            continue;
        }

        // ---- ... and the four waves (LDS): each hands over its state unscaled, and the reduction weights it ----
        // (The end of a segment is latency: ~2 ns for every instruction of a wave, a barrier for every hand-over.  One barrier instead of two -
        // the waves no longer scale to a common maximum first - 16-byte LDS stores and two channels a thread with each weight computed once;
        // us per call before / after: 16 users of 512-4096 + 1-512 tokens fused 31.66 / 31.18, token-major as two parties with the append
        // 42.01 / 41.32.  The slots it reads at once cost the two-step and paged instances 3-4 vector registers, within the same waves per
        // SIMD, and 2-5 spilled scalar ones: without them - an opaque copy of the thread's index here, as where NA is 1 - 400 random calls
        // take what they do with them.)
        int tid = threadIdx.x;
        if constexpr (NA == 1)
            asm("" : "+v"(tid));
        const int head = kQuad ? r & (kQuadHeads - 1) : r;  // the query head of the lane's results
        if (grp == 0)  // (4x4 blocks: entries past head 3 are copies, never read)
            sm_ml[wave][r] = make_float2(m, l);
        if constexpr (kQuad)
            reduce_scatter_groups<CP>(acc);
        if (head < G) {
            // rows 4*grp + v of the tile; 4x4 blocks: rows 4*rq + v, and of the phases the lane group's quarter
            float *dst = &sm_o[wave * o_wave_stride + head * kOStride];
            const int row0 = kQuad ? (r & ~3) : grp * 4, cc0 = kQuad ? (grp >> 1) * (CP / 2) + (grp & 1) * (CP / 4) : 0;
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
        __syncthreads();

        const int64_t head0 = (int64_t)it.user * Hq + (int64_t)it.kv_head * G;
        // the row goes to the ring - unless the piece ends here with an empty ring, or there is no ring
        const bool last = it.next < 0;
        const bool to_ring = ring_rows > 0 && !(last && n_ring == 0);
        const int GD = G * D, ring_stride = ring_row_floats(D, G);
        float *const ring = sm_o + kWaves * o_wave_stride;
        float *const dst_o = direct ? out + head0 * D : part_o + (int64_t)it.slot * GD;
        float *const dst_l = direct ? lse + head0 : part_lse + (int64_t)it.slot * G;
        // (two copies of the loop, so that each stores through pointers of one kind, LDS or global memory: a pointer
        // that may be either makes every store a flat one)
        typedef __attribute__((address_space(1))) float *global_f32;
        typedef __attribute__((address_space(3))) float *lds_f32;
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        auto reduce_waves = [&](auto row_o, auto row_l) {
            for (int idx = tid * 2; idx < GD; idx += kThreads * 2) {
                const int g = idx / D, ch = idx % D;
                float2 ml[kWaves];
                f32x2 x[kWaves];
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    ml[w] = sm_ml[w][g];
                    x[w] = *reinterpret_cast<const f32x2 *>(&sm_o[w * o_wave_stride + g * kOStride + ch]);
                }
                float M = ml[0].x;  // some wave holds tokens, so M is finite; an idle wave has m = -inf and weight 0
#pragma unroll
                for (int w = 1; w < kWaves; ++w)
                    M = fmaxf(M, ml[w].x);
                float o0 = 0.f, o1 = 0.f, lt = 0.f;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const float f = fast_exp2(ml[w].x - M);
                    o0 = fmaf(f, x[w][0], o0);
                    o1 = fmaf(f, x[w][1], o1);
                    lt = fmaf(f, ml[w].y, lt);
                }
                const float inv = fast_rcp(lt);
                row_o[idx] = o0 * inv;
                row_o[idx + 1] = o1 * inv;
                if (ch == 0)
                    row_l[g] = (M + fast_log2(lt) - Elt<DT>::kPShift) * kLn2;  // M is in log2 units
            }
        };
        if (to_ring)
            reduce_waves((lds_f32)(ring + n_ring * ring_stride), (lds_f32)(ring + n_ring * ring_stride + GD));
        else
            reduce_waves((global_f32)dst_o, (global_f32)dst_l);
        if (to_ring) {
            if (tid == 0) {
                ring_dst_o[n_ring] = dst_o;
                ring_dst_l[n_ring] = dst_l;
            }
            ++n_ring;
            if (last || n_ring == ring_rows) {
                __syncthreads();
                for (int i = 0; i < n_ring; ++i) {
                    const lds_f32 src = (lds_f32)(ring + i * ring_stride);
                    const global_f32 o = (global_f32)ring_dst_o[i];
                    for (int idx = tid; idx < GD; idx += kThreads)
                        o[idx] = src[idx];
                    if (tid < G)
                        ((global_f32)ring_dst_l[i])[tid] = src[GD + tid];
                }
                n_ring = 0;
            }
        }
        if (last)
            return;
        if (!PREFETCH) {
            nx = grown(nx, grow);
            begin_segment(nx, L, qB, tb, T0, P);
        }
        it = nx;
        __syncthreads();  // the LDS staging arrays are reused by the next segment
    }
}

}  // namespace spd
