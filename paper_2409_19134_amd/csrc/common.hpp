// Shared device-side declarations of the SPD decode-attention kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>

#include "../../include/spd.h"

namespace spd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x8 __attribute__((ext_vector_type(8)));

constexpr int kWaves = 4;            // waves per workgroup in the partial-attention kernels
constexpr int kThreads = kWaves * 64;
constexpr int kRowsMaxWaves = 12;    // waves of a whole-rows workgroup: three per SIMD, what a tile's registers allow
constexpr int kMaxGroup = 16;        // query heads per KV head the MFMA tile can hold
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// A global address as a kernel's own parameter (not in a struct): the runtime looks up the allocation of every parameter that is declared a
// pointer, on each launch (host time of three whole-rows and merge calls 9.95 us with pointers, 9.75 with these).  So the kernels that a step
// or call launches on its usual paths take addresses; finalize_step_kernel (rows of more than 32 chunks), the merge of more than two parts,
// the mass tracker and the uploads of a new schedule keep pointers.
typedef uintptr_t Address;
template <class T>
__device__ __forceinline__ T *global_pointer(Address a)
{
    return (T *)(T __attribute__((address_space(1))) *)a;
}

// A kernel's last parameter: its type, and where it lies among the kernel's arguments (each at the next multiple of its alignment).
template <class F>
struct LastParameter;
template <class... P>
struct LastParameter<void (*)(P...)> {
    static constexpr size_t place()
    {
        size_t end = 0, at = 0;
        ((at = (end + alignof(P) - 1) / alignof(P) * alignof(P), end = at + sizeof(P)), ...);
        return at;
    }
    static constexpr size_t at = place();
    typedef std::tuple_element_t<sizeof...(P) - 1, std::tuple<P...>> type;
};

// A kernel's head, 14 dwords that are preloaded, as the parameters that it travels in: vectors, each one parameter for the runtime to go
// through on a launch.  (One user's calls through two launches, which the host bounds, us with a parameter for every field / with three
// vectors / with one struct and nothing preloaded: 9.0 / 8.8 / 8.9, 8.8 / 8.7 / 8.7, fused 7.8 / 7.7 / 7.7.)
struct HeadWords {
    u32x8 a;
    u32x4 b;
    u32x2 c;
};
template <class Head>
__host__ __device__ __forceinline__ HeadWords head_words(const Head &h)
{
    static_assert(sizeof(Head) == 14 * 4, "the head is what the parameters hold");
    HeadWords w;
    __builtin_memcpy(&w.a, reinterpret_cast<const char *>(&h), sizeof w.a);
    __builtin_memcpy(&w.b, reinterpret_cast<const char *>(&h) + sizeof w.a, sizeof w.b);
    __builtin_memcpy(&w.c, reinterpret_cast<const char *>(&h) + sizeof w.a + sizeof w.b, sizeof w.c);
    return w;
}
template <class Head>
__device__ __forceinline__ Head head_of(u32x8 a, u32x4 b, u32x2 c)
{
    Head h;
    __builtin_memcpy(reinterpret_cast<char *>(&h), &a, sizeof a);
    __builtin_memcpy(reinterpret_cast<char *>(&h) + sizeof a, &b, sizeof b);
    __builtin_memcpy(reinterpret_cast<char *>(&h) + sizeof a + sizeof b, &c, sizeof c);
    return h;
}

// Addressing of one owner's cache; all strides in BYTES.  Base pointers travel in the work items.
struct KvAddr {
    const int32_t *block_table;  // paged mode only, else nullptr
    int32_t max_blocks;
    int32_t page_shift;  // paged mode: a page holds 1 << page_shift tokens (16 .. 256)
    int64_t block_stride;
    int64_t token_stride;
    int64_t head_stride;  // used by the head-per-wave kernel only (token-major storage: the same for every user)
};

// One segment of work as the kernels read it: tokens [t_begin, t_end) of one (user, KV head) row.  A workgroup
// processes a *piece*: a short list of segments linked by `next` (a piece that crosses a row boundary has one
// segment per row it touches).  k_base / v_base point at channel 0 of token 0 of the row (contiguous mode) or at the
// KV head's offset inside the pool (paged mode: a byte offset stored as a pointer, the pool base travels in OwnerArgs).  n_chunks == 0 marks a row without tokens: the workgroup only
// writes A = 0, lse = -inf.
struct DevItem {
    const char *k_base;
    const char *v_base;
    int32_t user, kv_head, t_begin, t_end;
    int32_t slot;      // where this segment's partial goes when the row has several segments (head-per-wave pieces:
                       // the slot of KV head 0; head h writes slot + h * n_chunks)
    int32_t n_chunks;  // segments of the row; 1: the segment writes the final result itself
    int32_t next;      // index of the piece's next segment, -1 if none
    int32_t rot;       // bits 0-1: 32-token steps the piece has already handed out (mod 4), keeps the four waves
                       // evenly loaded; bit 8 (kEndsRow): the segment ends at the last token of its row
};
constexpr int kEndsRow = 0x100;

// A (user, KV head) row of one owner as the whole-rows kernel reads it, indexed user * Hkv + KV head; addresses as in
// DevItem.
struct RowItem {
    const char *k_base, *v_base;
    int32_t t_end;  // tokens
    int32_t pad[3];
};

// 16-byte load of K/V data that is read exactly once: the non-temporal hint keeps the stream from displacing
// other lines in L2 (measured: plain streaming reads reach ~6.3 TB/s on this GPU, non-temporal ones ~7.1 TB/s).
// The pointer is cast to the global address space: base pointers arrive through memory (the work items), where the
// compiler cannot see the address space and would otherwise emit slower FLAT loads that also tie up the LDS counter.
template <typename V>  // V: u32x4 (16 bytes) or u32x2 (8 bytes)
__device__ __forceinline__ V stream_load(const char *p)
{
    typedef const V __attribute__((address_space(1))) *global_ptr;
    return __builtin_nontemporal_load((global_ptr)(uintptr_t)p);
}
__device__ __forceinline__ u32x4 stream_load16(const char *p) { return stream_load<u32x4>(p); }

// The same through a buffer descriptor over a row's tokens from tb to t_last, its last (rows of `bytes` bytes that lie end to end:
// offsets inside a step are small): a lane's offset from token tb.  What lies past the last token's row is zero; so is everything if
// tb does.  All of an offset is in the lane's part (and the instruction's immediate): those are what the range check is specified to
// cover, the scalar part is not.
typedef __amdgpu_buffer_rsrc_t row_rsrc;
__device__ __forceinline__ row_rsrc row_buffer(const char *row, int tb, int t_last, int64_t token_stride, int bytes)
{
    const int64_t left = (int64_t)(t_last - tb) * token_stride + bytes;
    const unsigned n = t_last < tb ? 0u : left > 0xffffffffll ? 0xffffffffu : (unsigned)left;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(row + (int64_t)tb * token_stride), 0, (int)n, 0x00020000);  // raw, no swizzle
}
constexpr int kBufferNonTemporal = 2;
__device__ __forceinline__ u32x4 stream_load16(row_rsrc b, unsigned at)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, kBufferNonTemporal));
}

// Wave-uniform values (work item fields arrive through vector loads): tell the compiler, so that address arithmetic
// and the block-table lookups go to the scalar unit.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const char *uniform(const char *p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char *>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ DevItem uniform(const DevItem &it)
{
    DevItem u;
    u.k_base = uniform(it.k_base);
    u.v_base = uniform(it.v_base);
    u.user = uniform(it.user);
    u.kv_head = uniform(it.kv_head);
    u.t_begin = uniform(it.t_begin);
    u.t_end = uniform(it.t_end);
    u.slot = uniform(it.slot);
    u.n_chunks = uniform(it.n_chunks);
    u.next = uniform(it.next);
    u.rot = uniform(it.rot);
    return u;
}

// A work item read through the scalar cache (items are constant during a launch, the index is wave-uniform): the
// fields land in scalar registers and cost no vector registers while they wait to be used.
typedef const uint32_t __attribute__((address_space(4))) *const_u32_ptr;
__device__ __forceinline__ DevItem scalar_load_item(const DevItem *items, int idx)
{
    static_assert(sizeof(DevItem) == 48, "DevItem is read as 12 dwords");
    const const_u32_ptr w = (const_u32_ptr)(uintptr_t)(items + idx);
    DevItem it;
    it.k_base = reinterpret_cast<const char *>(((uint64_t)w[1] << 32) | w[0]);
    it.v_base = reinterpret_cast<const char *>(((uint64_t)w[3] << 32) | w[2]);
    it.user = (int32_t)w[4];
    it.kv_head = (int32_t)w[5];
    it.t_begin = (int32_t)w[6];
    it.t_end = (int32_t)w[7];
    it.slot = (int32_t)w[8];
    it.n_chunks = (int32_t)w[9];
    it.next = (int32_t)w[10];
    it.rot = (int32_t)w[11];
    return it;
}

// Block-table entry read through the scalar cache (the table is constant during a launch and the index is
// wave-uniform): it neither waits behind the vector loads of the K/V stream nor delays them.
typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
__device__ __forceinline__ int scalar_load_i32(const int32_t *p, int idx)
{
    return ((const_i32_ptr)(uintptr_t)p)[idx];
}

// A user's base pointer from a device pointer table, as an integer to add to the item's offset (0 without a table).
// Scalar cache: the table is constant during a launch and the index wave-uniform.
typedef const uint64_t __attribute__((address_space(4))) *const_u64_ptr;
__device__ __forceinline__ uintptr_t user_base(const char *const *table, int user)
{
    return table ? (uintptr_t)((const_u64_ptr)(uintptr_t)table)[user] : 0;
}

__device__ __forceinline__ void copy16(char *dst, const char *src)
{
    *reinterpret_cast<u32x4 *>(dst) = *reinterpret_cast<const u32x4 *>(src);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// hardware log2 and reciprocal (1 ulp): the epilogues are latency, every library call in them is a dozen instructions
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Exchanges between the four 16-lane groups of a wave (lane ^ 16, lane ^ 32) without a trip through the LDS crossbar:
// v_permlane16_swap trades the odd 16-lane rows of its first operand for the even rows of its second, v_permlane32_swap
// the upper half of the first for the lower half of the second.  Fed the same value twice, the two results hold, in
// every lane, the lane's own value and its partner's (in one order or the other), which is all a max or a sum needs.
template <int MASK>
__device__ __forceinline__ void wave_xor_pair(float v, float &a, float &b)
{
    static_assert(MASK == 16 || MASK == 32, "lane groups are 16 lanes wide");
    const unsigned u = __float_as_uint(v);
    if constexpr (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    }
}
template <int MASK>
__device__ __forceinline__ float wave_xor_max(float v)
{
    float a, b;
    wave_xor_pair<MASK>(v, a, b);
    return fmaxf(a, b);
}
template <int MASK>
__device__ __forceinline__ float wave_xor_sum(float v)
{
    float a, b;
    wave_xor_pair<MASK>(v, a, b);
    return a + b;
}

// Rows without tokens (Theorem 1 with an empty part): A = 0, lse = -inf for the G heads of the row.
template <int D>
__device__ __forceinline__ void write_empty_row(const DevItem &it, int G, int Hq, float *out, float *lse)
{
    const int64_t head0 = (int64_t)it.user * Hq + (int64_t)it.kv_head * G;
    for (int idx = threadIdx.x; idx < G * D; idx += blockDim.x)
        out[head0 * D + idx] = 0.f;
    if ((int)threadIdx.x < G)
        lse[head0 + threadIdx.x] = -INFINITY;
}

// Everything a partial kernel needs to know about one owner's call, besides its items and their growth.  A launch serves one owner,
// or - for the fused decode step - both at once: workgroups [0, n0) take owner 0's pieces, the rest owner 1's.  First what a
// workgroup needs before its first tile.
struct OwnerArgs {
    // contiguous mode with device pointer tables: the items' k_base / v_base are byte offsets from k_ptrs[user] /
    // v_ptrs[user] (so that the schedule does not depend on the buffers' addresses); else nullptr
    const char *const *k_ptrs;
    const char *const *v_ptrs;
    KvAddr kv;
    const char *k_pool;  // paged mode: the items' k_base / v_base are byte offsets inside these; else nullptr
    const char *v_pool;
    // KV append (protocol step 3a), or nullptr: [U][Hkv][D] rows of the new token's K and V.  The row's last token
    // (position lens[u] - 1) is then taken from here, and the segment that ends the row also writes it to the cache.
    const char *k_new;
    const char *v_new;
    float *out;       // [U][Hq][D]
    float *lse;       // [U][Hq]
    float *part_o;    // [slots][G][D] chunk partials of split rows
    float *part_lse;  // [slots][G]
};

// A work item with the row's growth applied.
__device__ __forceinline__ DevItem grown(DevItem it, int grow)
{
    it.t_end += (it.rot & kEndsRow) ? grow : 0;
    return it;
}

// A row (user, KV head) whose tokens were split into several chunks.
struct CombineRow {
    int32_t first_slot, n_chunks, user, kv_head;
};

// Chunk bookkeeping of every (user, KV head) row, indexed user * Hkv + kv_head.
struct RowInfo {
    int32_t first_slot, n_chunks;
};

// The partial kernel's arguments.  The head arrives in scalar registers with the wave (kernel-argument preloading: up to 14 dwords, not
// out of a struct), so that a workgroup's first instructions ask for its item; the owners are the last parameter, read at the one that the
// workgroup serves.
struct PartialHead {
    const DevItem *items[2];
    const char *q;          // [U][Hq][D]
    int32_t n0;             // workgroups [0, n0) serve owner 0, the rest owner 1
    // Tokens every row has gained since the schedule was built (a decode loop appends one token per user and step):
    // added to t_end of the segments that end their row, so that a schedule serves several consecutive steps.
    int32_t grow[2];
    int32_t Hq, G;
    float scale_log2e;
    int32_t ring_rows;      // result rows a workgroup may hold back in LDS (see the result ring in partial_mfma.hpp); 0: none
};
struct PartialArgs {
    OwnerArgs owner[2];
};
constexpr int kPartialArgsAt = sizeof(PartialHead);  // in the kernel's arguments (the launch checks it against the kernel's own parameters)
}  // namespace spd
