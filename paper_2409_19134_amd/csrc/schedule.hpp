// The split schedule of a partial-attention launch (host only, no HIP calls).
#pragma once
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <vector>

#include "../../include/spd.h"
#include "common.hpp"

namespace spd::host {

constexpr int kChunkAlign = 32;      // chunk boundaries are multiples of the MFMA kernel's 32-token step
constexpr int kChunkMin = 128;       // one 32-token step for each of the four waves
constexpr int kShortPieceSteps = 64;  // 32-token steps per piece up to which Tuning::seg_cost and half_skew apply
// (32-token steps * KV heads) per CU from which the head-per-wave mapping is used, and from which its workgroups take
// eight heads instead of four (see head_per_wave_choice in spd_api.hip)
constexpr int kHeadPerWaveMinHeadSteps = 65;
constexpr int kHeadPerWaveMinHeadSteps64 = 40, kHeadPerWaveMinHeadSteps64OneOwner = 32, kHeadPerWaveMinHeadStepsOneOwner = 41;
constexpr int kHeadPerWaveWideHeadSteps = 900;
constexpr int kHeadPerWaveWideHeadStepsMany = 340;  // more than eight KV heads

// What shapes a schedule besides the lengths.  A context starts from the defaults below, replaced by SPD_* variables
// of the environment that spd_create finds set (tuning_from_env), and spd_set_option changes them per context; all
// of them are part of the key a cached schedule is remembered by.
struct Tuning {
    // workgroups of the MFMA kernel resident per CU (2 waves per SIMD)                        SPD_TARGET_WG_PER_CU
    int32_t target_wg_per_cu = 2;
    // if no row is longer than this the work is latency-bound: every row is cut into chunks of one step per wave
    //                                                                                          SPD_NO_SPLIT_MAX
    int32_t no_split_max = 768;
    // tokens per piece when the work exceeds one resident round: a new workgroup costs a few microseconds of an idle
    // slot, more than the longer tail of bigger pieces (4096: 3 % slower on the longest workload)  SPD_CHUNK_MAX
    int32_t chunk_max = 16384;
    // 32-token steps a piece gives up for every further row it reaches into (a second segment costs an epilogue and a
    // memory round trip before the new row's first tile; measured on the headline workload: 0 -> 2 steps takes
    // 0.45 us off a 32.5 us step, 4 and more give it back)                                      SPD_SEG_COST
    int32_t seg_cost = 2;
    // When the pieces are exactly one resident round, the half dispatched first gets (100 + s) % of the mean piece and
    // the other half (100 - s) %: every workgroup asks for its first tile in the same microsecond, the memory system
    // serves those ~35 MB in launch order, and the half served last stays ~4 us behind to the end (measured with
    // in-kernel time stamps); unequal shares let both halves finish together (0 -> 12 %: -0.35 us)  SPD_HALF_SKEW
    int32_t half_skew = 12;
};
constexpr int kTuningInts = 5;
static_assert(sizeof(Tuning) == kTuningInts * sizeof(int32_t), "the key takes the struct as kTuningInts integers");

inline int env_int(const char *name, int dflt, int least = 1)
{
    const char *s = std::getenv(name);
    if (!s || !*s)
        return dflt;
    const long v = std::strtol(s, nullptr, 10);
    return v >= least && v <= (1 << 30) ? (int)v : dflt;
}

inline Tuning tuning_from_env()
{
    Tuning t;
    t.target_wg_per_cu = env_int("SPD_TARGET_WG_PER_CU", t.target_wg_per_cu);
    t.no_split_max = env_int("SPD_NO_SPLIT_MAX", t.no_split_max);
    t.chunk_max = env_int("SPD_CHUNK_MAX", t.chunk_max);
    t.seg_cost = env_int("SPD_SEG_COST", t.seg_cost, 0);
    t.half_skew = std::min(90, env_int("SPD_HALF_SKEW", t.half_skew, 0));
    return t;
}

// The split schedule ("stream-K" over tokens), for calls whose rows are not taken whole (whole_rows_choice).
// All KV heads of a user hold the same tokens, so the schedule is laid
// out on token steps (32 tokens) per user and replicated over the KV heads: the steps of all users, laid end to end,
// are divided into groups of equal length (+-1 step), and every group becomes one piece (one workgroup) per KV head.
// The pieces of a group are adjacent in launch order, so with token-major storage the heads that share DRAM pages
// stream them at the same time.  A group that crosses a user boundary gives pieces with several segments.
// Equal pieces matter because the path is HBM-bound: a launch lasts as long as its longest workgroup.
//   - if no user is longer than a few hundred tokens the work is latency-bound: every row is cut into chunks of 128
//     tokens (one step per wave: one memory round trip), also for a standalone call, although it then needs the combine
//     launch (rows that pay for being whole are taken by the whole-rows kernel instead);
//   - work that fits one resident wave of workgroups (2 per CU) gets exactly that many pieces;
//   - larger work gets pieces of at most `piece_max` tokens, their number rounded up to a multiple of the resident
//     wave, and relies on the hardware's dynamic workgroup dispatch.
struct Schedule {
    std::vector<spd_work_item> items;  // segments in piece order (rows with tokens only)
    std::vector<int32_t> piece_first;  // [n_pieces + 1] first segment of each piece
    int64_t n_slots = 0;
    int chunk_tokens = 0;              // tokens per piece (rounded up)
};

// hpw: pieces for the head-per-wave kernel (token-major storage).  A piece then covers all KV heads of its token
// range (a group of up to eight of them, see head_per_wave_waves): one item per cut and group (kv_head and slot are
// those of the group's first head) and one resident workgroup per CU.  The same
// token limit per piece serves both mappings (smaller pieces measured slower here too), although every wave now
// walks the whole range instead of a quarter of it.
// Waves (KV heads) per workgroup of the head-per-wave mapping: the largest divisor of Hkv that is at most `most`
// (8: two waves per SIMD is what the kernel's registers allow); Hkv / that many head groups share a token range.
inline int head_per_wave_waves(int Hkv, int most = 8)
{
    for (int w = std::min(Hkv, std::min(most, 8)); w >= 1; --w)
        if (Hkv % w == 0)
            return w;
    return 1;
}

// The number of pieces build_schedule makes for the head-major mapping if they are exactly one resident round of
// equal pieces (target_wg_per_cu per CU), else 0 (short rows cut into one-step chunks, less work than a round, or
// several rounds).  Costs a pass over the lengths: the fused step asks before it looks its schedules up.
// *rows: the (user, KV head) rows that hold tokens; *steps (if asked for): the 32-token steps of one KV head.
inline int64_t single_round_pieces(int Hkv, int n_users, const int32_t *lens, int n_cus, const Tuning &tune, int64_t *rows,
                                   int64_t *steps_out = nullptr)
{
    int64_t T = 0, short_chunks = 0;
    int max_len = 0;
    *rows = 0;
    for (int u = 0; u < n_users; ++u) {
        const int64_t steps = (lens[u] + kChunkAlign - 1) / kChunkAlign;
        T += steps;
        short_chunks += (steps + spd::kWaves - 1) / spd::kWaves;
        max_len = std::max(max_len, lens[u]);
        *rows += lens[u] > 0 ? Hkv : 0;
    }
    if (steps_out)
        *steps_out = T;
    const int64_t resident = (int64_t)std::max(1, n_cus) * tune.target_wg_per_cu;
    if (T == 0 || (max_len <= tune.no_split_max && short_chunks * Hkv <= resident))
        return 0;
    const int64_t wg = std::max<int64_t>(1, resident / Hkv);
    const int64_t piece_max = std::max(kChunkMin, (int)tune.chunk_max) / kChunkAlign;
    if (T > wg * piece_max || (T + spd::kWaves - 1) / spd::kWaves < wg)
        return 0;
    return wg * Hkv;
}

// hpw: 0 for the head-major mapping, else the KV heads (waves) per workgroup of the head-per-wave mapping, a divisor
// of Hkv that is at most 8.
inline void build_schedule(int Hkv, int n_users, const int32_t *lens, int n_cus, int hpw, const Tuning &tune, Schedule &S)
{
    const int hpw_waves = hpw ? hpw : 1;
    const int hpw_groups = hpw ? Hkv / hpw_waves : 1;
    S.items.clear();
    S.piece_first.assign(1, 0);
    S.n_slots = 0;
    S.chunk_tokens = 0;
    int64_t T = 0;  // total 32-token steps per KV head
    int max_len = 0;
    for (int u = 0; u < n_users; ++u) {
        T += (lens[u] + kChunkAlign - 1) / kChunkAlign;
        max_len = std::max(max_len, lens[u]);
    }
    if (T == 0)
        return;

    // a group: user-local step ranges; cut[g] lists (user, first step, end step)
    struct Cut {
        int user;
        int64_t s0, s1;
    };
    std::vector<std::vector<Cut>> groups;
    // Short rows are cut into chunks of one step per wave - unless that makes more workgroups than fit the machine
    // at once: many users with short rows are bandwidth-bound like any large launch and get equal pieces instead
    // (measured, 64 users x <= 512 + 256 tokens, 117 MB: 31.7 us against 35.6 us per fused step).
    int64_t short_chunks = 0;
    for (int u = 0; u < n_users; ++u)
        short_chunks += ((lens[u] + kChunkAlign - 1) / kChunkAlign + spd::kWaves - 1) / spd::kWaves;
    const int64_t resident = (int64_t)std::max(1, n_cus) * tune.target_wg_per_cu;
    if (max_len <= tune.no_split_max && short_chunks * (hpw ? hpw_groups : Hkv) <= resident) {
        const int64_t per = spd::kWaves;  // steps per chunk
        for (int u = 0; u < n_users; ++u) {
            const int64_t steps = (lens[u] + kChunkAlign - 1) / kChunkAlign;
            for (int64_t s0 = 0; s0 < steps; s0 += per)
                groups.push_back({Cut{u, s0, std::min(steps, s0 + per)}});
        }
        S.chunk_tokens = (int)std::min<int64_t>(per, (max_len + kChunkAlign - 1) / kChunkAlign) * kChunkAlign;
    } else {
        const int64_t slots = resident;
        // groups per resident wave of workgroups
        // head per wave: a CU holds eight such waves, i.e. 8 / waves workgroups
        const int64_t wg = hpw ? std::max<int64_t>(1, (int64_t)std::max(1, n_cus) * (8 / hpw_waves) / hpw_groups)
                               : std::max<int64_t>(1, slots / Hkv);
        const int64_t piece_max = std::max(kChunkMin, (int)tune.chunk_max) / kChunkAlign;
        // group boundaries (cumulative step counts)
        std::vector<int64_t> ends;
        std::vector<int64_t> cut_num;  // group i ends at the fraction cut_num[i] / cut_den of the line
        int64_t cut_den = 1;
        if (T <= wg * piece_max) {
            // at least one step per wave
            // (measured on the headline workload: fewer, round-aligned pieces or more pieces than fit at once are
            // both slower - 55 groups of 20 steps +2 us, 80 groups +1.5 us against 64 groups of 17-18 steps)
            const int64_t W = std::min<int64_t>(wg, hpw ? T : (T + spd::kWaves - 1) / spd::kWaves);
            // exactly one resident round of head-major pieces of 8 to kShortPieceSteps steps: unequal halves (see Tuning;
            // the ~4 us by which the second half trails do not matter to longer pieces: workload 4, 214 steps, +0.2 %)
            const int64_t skew = (!hpw && W == wg && W >= 2 && T >= 8 * W && T <= kShortPieceSteps * W) ? tune.half_skew : 0;
            for (int64_t i = 0; i < W; ++i) {
                const int64_t h = W / 2;
                // cumulative weight up to group i (inclusive), in percent-groups
                const int64_t cum = (i + 1 <= h) ? (i + 1) * (100 + skew) : h * (100 + skew) + (i + 1 - h) * (100 - skew);
                const int64_t tot = h * (100 + skew) + (W - h) * (100 - skew);
                ends.push_back(T * cum / tot);
                cut_num.push_back(cum);
                cut_den = tot;
            }
        } else {
            // several resident waves of equal pieces; the hardware hands them out in launch order.  (Cutting the last
            // wave's share finer to shorten the tail was measured and lost 1-3 %: short pieces cost more than the tail.)
            const int64_t W = wg * ((T + wg * piece_max - 1) / (wg * piece_max));
            for (int64_t i = 0; i < W; ++i) {
                ends.push_back(T * (i + 1) / W);
                cut_num.push_back(i + 1);
            }
            cut_den = W;
        }
        // A piece that crosses into another user's row pays for a second segment (an epilogue, and a memory round
        // trip before the new row's first tile): such pieces get `seg_cost` steps fewer.  The cuts are made on a line
        // that holds seg_cost extra steps in front of every user but the first; a cut that lands in such a gap moves
        // to the user's boundary.
        // Only for pieces of up to kShortPieceSteps steps: measured, 2 steps take 1.4 % off the headline workload's step
        // (pieces of 17 steps) and 3 % off 256 users with 64-512-token rows (36 steps), but add 0.9 % to workload 4
        // (pieces of 214 steps over four rows each), where the unequal lengths cost more than the segments.
        const int64_t seg_cost = T <= kShortPieceSteps * (int64_t)ends.size() ? tune.seg_cost : 0;
        if (seg_cost > 0) {
            int64_t n_rows_with_tokens = 0;
            for (int u = 0; u < n_users; ++u)
                n_rows_with_tokens += lens[u] > 0;
            const int64_t Tv = T + seg_cost * std::max<int64_t>(0, n_rows_with_tokens - 1);
            size_t i = 0;
            int64_t real0 = 0, virt0 = 0;  // the current user's first step on the real and on the stretched line
            bool first = true;
            for (int u = 0; u < n_users && i < ends.size(); ++u) {
                const int64_t steps = (lens[u] + kChunkAlign - 1) / kChunkAlign;
                if (steps == 0)
                    continue;
                if (!first)
                    virt0 += seg_cost;
                first = false;
                // cuts (on the stretched line) up to the end of this user's steps
                while (i < ends.size()) {
                    const int64_t cut = Tv * cut_num[i] / cut_den;
                    if (cut > virt0 + steps)
                        break;
                    ends[i++] = real0 + std::max<int64_t>(0, cut - virt0);
                }
                real0 += steps;
                virt0 += steps;
            }
            for (; i < ends.size(); ++i)
                ends[i] = T;
            ends.back() = T;
        }
        const int64_t W = (int64_t)ends.size();
        int64_t longest = ends[0];
        for (size_t i = 1; i < ends.size(); ++i)
            longest = std::max(longest, ends[i] - ends[i - 1]);
        S.chunk_tokens = (int)longest * kChunkAlign;
        groups.resize((size_t)W);
        int64_t g0 = 0;  // global step index of the current user's first step
        int64_t g = 0;
        for (int u = 0; u < n_users; ++u) {
            const int64_t steps = (lens[u] + kChunkAlign - 1) / kChunkAlign;
            int64_t s = 0;
            while (s < steps) {
                while (ends[(size_t)g] <= g0 + s)
                    ++g;
                const int64_t e = std::min(steps, ends[(size_t)g] - g0);
                groups[(size_t)g].push_back(Cut{u, s, e});
                s = e;
            }
            g0 += steps;
        }
    }

    // chunks per user (same for all its KV heads) and the first partial slot of every row
    std::vector<int32_t> n_chunks((size_t)n_users, 0), seen((size_t)n_users, 0);
    for (const auto &grp : groups)
        for (const Cut &c : grp)
            ++n_chunks[(size_t)c.user];
    std::vector<int64_t> user_slot0((size_t)n_users, 0);
    for (int u = 0; u < n_users; ++u) {
        user_slot0[(size_t)u] = S.n_slots;
        S.n_slots += (int64_t)n_chunks[(size_t)u] * Hkv;
    }
    int32_t piece = 0;
    for (const auto &grp : groups) {
        if (grp.empty())
            continue;
        for (int hh = 0; hh < (hpw ? hpw_groups : Hkv); ++hh) {
            const int h = hpw ? hh * hpw_waves : hh;  // head per wave: the first head of the group
            for (const Cut &c : grp) {
                spd_work_item it;
                it.user = c.user;
                it.kv_head = h;
                it.t_begin = (int32_t)(c.s0 * kChunkAlign);
                it.t_end = (int32_t)std::min<int64_t>(lens[c.user], c.s1 * kChunkAlign);
                it.n_chunks = n_chunks[(size_t)c.user];
                it.chunk = seen[(size_t)c.user];
                it.slot = (int32_t)(user_slot0[(size_t)c.user] + (int64_t)h * it.n_chunks + it.chunk);
                it.piece = piece;
                S.items.push_back(it);
            }
            ++piece;
            S.piece_first.push_back((int32_t)S.items.size());
        }
        for (const Cut &c : grp)
            ++seen[(size_t)c.user];
    }
}

// What the kernels read of a schedule, as it is laid out in device memory.
struct DeviceTables {
    std::vector<spd::DevItem> items;          // [items_launched] first segments and empty rows, then the continuation segments
    std::vector<spd::CombineRow> split_rows;  // rows held in more than one partial slot
    std::vector<spd::RowInfo> row_info;       // [n_users * Hkv] first slot and slot count of every row
    int64_t items_launched = 0;               // workgroups of the launch
    int64_t n_segments = 0;                   // segments with tokens, all pieces together
};

// The address of row (user, KV head h) of a view - or, where the kernel adds the pool or the user's pointer itself, its
// offset from that.  es: bytes per K/V element.
inline const char *row_base(const spd_kv_view *v, int es, int u, int h, bool is_v)
{
    const uintptr_t base = (v->block_size || v->k_ptrs_dev) ? 0 : reinterpret_cast<uintptr_t>(is_v ? v->v_ptrs[u] : v->k_ptrs[u]);
    const int64_t hs = (v->head_strides && v->block_size == 0) ? v->head_strides[u] : v->head_stride;
    return reinterpret_cast<const char *>(base + (uintptr_t)((int64_t)h * hs * es));
}

// The tables of the whole-rows kernel: an item per row, indexed user * Hkv + KV head, and the users by length, longest
// first (the launch order where the rows do not all fit the device at once).
constexpr int kWholeRows = 64;  // in place of the head-per-wave mapping's KV heads per workgroup (0, 2..8)
// As laid out for device memory: RowItem[n_users * Hkv] | int32[n_users], each part 256-byte aligned.
inline size_t whole_rows_order_offset(int n_users, int Hkv)
{
    return ((size_t)n_users * Hkv * sizeof(spd::RowItem) + 255) / 256 * 256;
}
inline size_t whole_rows_bytes(int n_users, int Hkv)
{
    return whole_rows_order_offset(n_users, Hkv) + ((size_t)n_users * sizeof(int32_t) + 255) / 256 * 256;
}
inline void build_whole_rows(int Hkv, int es, const spd_kv_view *v, std::vector<spd::RowItem> &items, std::vector<int32_t> &order)
{
    items.assign((size_t)v->n_users * Hkv, spd::RowItem{});
    order.resize((size_t)v->n_users);
    for (int u = 0; u < v->n_users; ++u) {
        order[(size_t)u] = u;
        for (int h = 0; h < Hkv && v->lens[u] > 0; ++h) {
            spd::RowItem &d = items[(size_t)u * Hkv + h];
            d.k_base = row_base(v, es, u, h, false);
            d.v_base = row_base(v, es, u, h, true);
            d.t_end = v->lens[u];
        }
    }
    std::stable_sort(order.begin(), order.end(), [v](int32_t a, int32_t b) { return v->lens[a] > v->lens[b]; });
}

// Whether the rows of a whole-rows launch are started by length, longest first: there are more of them than workgroups of that
// many waves (of the twelve that fit a compute unit) are resident at once.
inline bool whole_rows_by_length(int64_t rows, int waves, int n_cus)
{
    return rows > (int64_t)std::max(1, n_cus) * (spd::kRowsMaxWaves / waves);
}

// Whether a call's rows are taken whole, one workgroup each, and by how many waves.  In units of 16 KB (a wave's step; with
// rows of 128 bytes two steps): `longest` is the longest row, `share` what each of the workgroups resident at once gets if the
// rows spread evenly.  Against the split schedule a whole-rows launch saves the closing launch and the ends of segments inside
// a piece, and loses what the device idles while its last rows end.  Where the lines lie was measured on 540 random calls over
// all layouts, element types and head groupings (1 to 256 users, rows of up to 90 units, appends, fused steps and one owner's
// calls), split against whole; us per call, 256 units:
//  - a unit for every row (rows <= units): the longest row's excess over the share, 0.3-0.5 us a unit, against 3-5 us.  Fused
//    steps 13.2 / 8.7 (excess 2), 18.9 / 17.5 (11), 18.0 / 17.4 (14), 17.2 / 19.5 (20); 14.7 / 16.6 (16); 10.5 / 12.2 (14).  One
//    owner's call saves less: 13.2 / 11.8 (9.6), 13.2 / 13.9 (11), 13.8 / 15.3 (12.4).
//    With a few rows (up to an eighth of the units), 1 and 4 users: 8.6 / 7.9 and 8.7 / 8.4 (14), 8.3 / 8.6 and 8.7 / 9.3 (16), with
//    the append in pages 8.7 / 8.2 and 8.7 / 8.6 (13), 8.6 / 9.3 (4 users, 14); rows of 128 bytes 8.5 / 7.5 (11), 8.8 / 9.0 (14),
//    with the append in pages 8.5 / 8.7 and 8.6 / 10.3; fp32 10.0 / 9.2 (14), 9.2 / 11.0 (7 heads, 15.5).  One owner's call up
//    to 16, where it is even on the device (8.9 / 8.9) and a caller that the host's launches bound saves 3 us (from Python 11.7 /
//    8.4), fp32 8.9 / 9.9 (15.4).  Rows of 128 bytes in general 9.8 / 9.7 (one owner, 7), 13.4 / 14.1 (8).
//  - up to two rows a unit and more than 16 steps: two rounds of one eight-wave workgroup per unit.  With half of the second
//    round empty the first one's saving is lost: 30.9 / 33.1 (320 rows), 54.0 / 71.5 (304), 25.5 / 28.5 (272), 24.0 / 25.1
//    (400); 33.1 / 32.2 (432), 50.5 / 48.7 (496), 34.7 / 30.2 (512); and with long rows there is nothing left to save, 84.4 / 88.0
//    (512 of 63 units), 51.0 / 51.7 (424 of up to 64).  With up to 16 steps four waves a row, all resident: 18.2 / 14.7 (376).
//  - more, up to three a unit: all resident, four waves a row, which cannot take in more than a wave's step at a time: the
//    excess counts more.  42.6 / 37.1 (3.1), 86.8 / 82.2 (2.3); 41.4 / 42.4 (6.5), 39.9 / 44.1 (12.7), 32.1 / 37.2 (20).  Rows of
//    128 bytes 22.1 / 20.3 (5), 51.5 / 56.4 (7.5).  With rows of up to 16 units only the start and the end count: 27.3 / 25.0 (5.6).
//  - more: the shortest rows come last.  If they are long and the last round is nearly empty, the device idles for them: 856 rows
//    of 56 units 132.9 / 136.7, 932 of 49 122.1 / 122.7; 1160 of 25 86.5 / 87.1, 840 of 16 43.6 / 39.2, 1044 of 36
//    112.7 / 108.0; of mixed lengths 936 rows of 15-33 97.4 / 90.7, 1016 of 4-35 67.8 / 59.4, 1872 of 2-18 70.0 / 49.7.
//  - token-major storage that the head-per-wave mapping would take (it reads a token's heads, whole DRAM pages, together): only
//    short rows, 35.9 / 28.7 (13 units), 54.2 / 44.5 (8), 33.5 / 38.0 (17), 60.5 / 68.8 (25), 59.7 / 78.6 (61) - and longer ones
//    where 256-byte rows fill several rounds, 130.4 / 116.1 (two parties, 2048 rows of up to 24; of 128 bytes, 1696 of up to 20,
//    111.4 / 125.0).
//  - rows of more than 64 units (2048 tokens at 256 bytes) gain nothing on balanced launches (256 users of 500-4000 + 1000:
//    454 / 477), fp32 rows of 512 bytes from 48 (56.3 / 57.4 at 58).
// The figures are of the kernels that placed the lines; both sides have got faster since (split calls by 0.5-1.4 us, whole ones by 0.2-0.6).
// 600 further random calls with both as they are now (profiles/whole_rows_rule_calls_timed.txt): of 362 that the rule takes whole 21 are
// more than 3 % faster split (51 us in all against 1166 gained) - few users at 12 to 14 steps 8.6 / 7.6, 10.0 / 8.2, 64 channels token-major
// 41.8 / 34.5, 49.5 / 44.6 - and of 44 up to 5 units beyond the lines 5 would be more than 3 % faster whole, 32 slower.
struct WholeRowsLoad {
    int tile = 32, step_bytes = 16384;  // tokens and K/V bytes of a wave's step
    int Hkv = 0, n_cus = 0, n_users = 0;
    int head_channels = 0;  // result channels of a row: query heads per KV head * channels
    const int32_t *lens0 = nullptr, *lens1 = nullptr;  // lens1: the second owner's, or nullptr
    bool f32 = false;
    bool always = false;  // whole rows whatever the rule says: the wave count is all that is asked for
};
constexpr int kWholeRowsLimit = 64, kWholeRowsLimit512 = 48, kWholeRowsLimitTwoRounds = 40;  // longest row
constexpr int kWholeRowsLimitTokenMajor = 16, kWholeRowsLimitTokenMajorMany = 32;  // (many: two full rounds)
constexpr int kWholeRowsTail = 12, kWholeRowsTailOneOwner = 10, kWholeRowsTail128 = 7;  // excess over the share
constexpr int kWholeRowsTailFew = 14, kWholeRowsTailFew128 = 11;
constexpr int kWholeRowsTailFewOneOwner = 16, kWholeRowsTailFewOneOwnerF32 = 13;
constexpr int kWholeRowsTailOneRound = 6, kWholeRowsTailOneRound128 = 5, kWholeRowsTailOneRoundShort = 8;
constexpr int kWholeRowsShort = 5;    // rows that are taken whole whatever their number
// head_per_wave(steps): whether the head-per-wave mapping would take a call of that many 32-token steps.
template <class F>
inline int whole_rows_choice(const WholeRowsLoad &c, F &&head_per_wave)
{
    // (one pass over the lengths per call: a step's tokens are a power of two, and the steps of two lengths of at most 2^30 tokens
    // fit 32 bits)
    const int shift = __builtin_ctz((unsigned)c.tile), up = c.tile - 1;
    int32_t longest_row = 0, shortest_row = INT32_MAX;
    int64_t total = 0;  // steps
    auto take = [&](int32_t steps) {
        longest_row = std::max(longest_row, steps);
        shortest_row = std::min(shortest_row, steps);
        total += steps;
    };
    if (c.lens1)
        for (int u = 0; u < c.n_users; ++u)
            take(((c.lens0[u] + up) >> shift) + ((c.lens1[u] + up) >> shift));
    else
        for (int u = 0; u < c.n_users; ++u)
            take((c.lens0[u] + up) >> shift);
    const int64_t longest = longest_row, shortest = shortest_row;
    const int64_t rows = (int64_t)c.n_users * c.Hkv, cus = std::max(1, c.n_cus), unit = 16384;
    const int row_bytes = c.step_bytes / (2 * c.tile);
    // Waves: twelve fit a compute unit, whatever the workgroups.  Rows that all have a unit of their own take as few waves
    // as make the same number of rounds; up to two rows per unit, eight waves (one workgroup per unit and a second round)
    // from 17 steps on and four below (64 users of <= 768 + 256 tokens 30.1 / 32.0 us, of <= 192 + 64 12.0 / 11.0); more
    // rows, four waves (256 users of <= 512 + 256 tokens: 82 us, 94 with eight or twelve).
    const bool two_rounds = rows > cus && rows <= 2 * cus && longest > 16;
    int64_t waves = 4, slots = 3 * cus;
    if (rows <= cus) {
        const int64_t rounds = std::max<int64_t>(1, (longest + spd::kRowsMaxWaves - 1) / spd::kRowsMaxWaves);
        waves = std::max<int64_t>(1, (longest + rounds - 1) / rounds);
        slots = cus;
    } else if (two_rounds) {
        waves = 8;
        slots = cus;
    }
    if (!c.always) {
        int64_t limit = row_bytes == 512 ? kWholeRowsLimit512 : kWholeRowsLimit;
        if (head_per_wave(total))
            limit = rows >= 2 * slots && row_bytes > 128 ? kWholeRowsLimitTokenMajorMany : kWholeRowsLimitTokenMajor;
        if (two_rounds)
            limit = std::min<int64_t>(limit, kWholeRowsLimitTwoRounds);
        int64_t tail = row_bytes == 128 ? kWholeRowsTail128 : c.lens1 ? kWholeRowsTail : kWholeRowsTailOneOwner;
        if (rows * 8 <= cus)
            tail = c.lens1 ? (row_bytes == 128 ? kWholeRowsTailFew128 : kWholeRowsTailFew)
                           : (c.f32 ? kWholeRowsTailFewOneOwnerF32 : kWholeRowsTailFewOneOwner);
        else if (rows > 2 * cus && rows <= slots)
            tail = longest * c.step_bytes <= 16 * unit ? kWholeRowsTailOneRoundShort
                   : row_bytes == 128                  ? kWholeRowsTailOneRound128
                                                       : kWholeRowsTailOneRound;
        if (longest * c.step_bytes > limit * unit || longest * c.step_bytes - total * c.Hkv * c.step_bytes / slots > tail * unit)
            return 0;
        if (two_rounds && 16 * rows <= 25 * cus && longest * c.step_bytes > kWholeRowsShort * unit)
            return 0;
        // the part of the last round that is empty, in slots, times the shortest row
        const int64_t empty = (slots - rows % slots) % slots;
        if (rows > 2 * cus && rows > slots && shortest * c.step_bytes * empty > 16 * unit * slots)
            return 0;
    }
    // No more waves than the longest row has steps - but up to four for the reduction of many result channels, whatever the
    // steps (a thread takes four channels at a time; 16 query heads of 128 channels, one step: 6.3 us per call, with four waves 4.2,
    // split 4.7; 8 heads 4.9 / 3.7 / 4.3).
    return (int)std::max(std::min(waves, std::max<int64_t>(1, longest)), std::min<int64_t>(4, (c.head_channels + 255) / 256));
}

// es: bytes per K/V element.  Row addresses come from the view's host pointer arrays (contiguous mode without device
// pointer tables); in the other modes the items hold offsets and the kernel adds the pool or the user's pointer.
inline void build_device_tables(const Schedule &S, int Hkv, int es, const spd_kv_view *v, int hpw, DeviceTables &T)
{
    using spd::CombineRow;
    using spd::DevItem;
    using spd::RowInfo;
    // device items: the first segment of every piece (index = workgroup id), then one per row without tokens (it only
    // writes A = 0, lse = -inf), then the continuation segments, linked through `next`
    const int hpw_waves = hpw ? hpw : 1;  // heads an item stands for
    const int64_t n_pieces = (int64_t)S.piece_first.size() - 1;
    int64_t n_empty_rows = 0;  // workgroups that only write A = 0, lse = -inf (head-per-wave: one per empty user)
    for (int u = 0; u < v->n_users; ++u)
        n_empty_rows += v->lens[u] == 0 ? (hpw ? Hkv / hpw_waves : Hkv) : 0;
    const int64_t n_groups = n_pieces + n_empty_rows;  // launched workgroups
    std::vector<DevItem> &dev_items = T.items;
    dev_items.assign((size_t)n_groups, DevItem{});
    dev_items.reserve((size_t)n_groups + S.items.size());
    auto to_dev = [&](const spd_work_item &w, int rot) {
        DevItem d;
        const int h = hpw ? 0 : w.kv_head;  // head per wave: every wave adds its own head's offset (from head 0)
        d.k_base = row_base(v, es, w.user, h, false);
        d.v_base = row_base(v, es, w.user, h, true);
        d.user = w.user;
        d.kv_head = w.kv_head;
        d.t_begin = w.t_begin;
        d.t_end = w.t_end;
        d.slot = w.slot;
        d.n_chunks = w.n_chunks;
        d.next = -1;
        d.rot = (rot & (spd::kWaves - 1)) | (w.t_end == v->lens[w.user] ? spd::kEndsRow : 0);
        return d;
    };
    for (int64_t pc = 0; pc < n_pieces; ++pc) {
        int rot = 0;
        size_t prev = 0;
        for (int32_t i = S.piece_first[(size_t)pc]; i < S.piece_first[(size_t)pc + 1]; ++i) {
            const spd_work_item &w = S.items[(size_t)i];
            const DevItem d = to_dev(w, rot);
            size_t at;
            if (i == S.piece_first[(size_t)pc]) {
                at = (size_t)pc;
                dev_items[at] = d;
            } else {
                at = dev_items.size();
                dev_items.push_back(d);
                dev_items[prev].next = (int32_t)at;
            }
            prev = at;
            rot += (w.t_end - w.t_begin + kChunkAlign - 1) / kChunkAlign;
        }
    }
    {
        size_t at = (size_t)n_pieces;
        for (int u = 0; u < v->n_users; ++u) {
            if (v->lens[u] != 0)
                continue;
            for (int hh = 0; hh < (hpw ? Hkv / hpw_waves : Hkv); ++hh) {
                DevItem d;
                d.k_base = d.v_base = nullptr;
                d.user = u;
                d.kv_head = hpw ? hh * hpw_waves : hh;
                d.t_begin = d.t_end = 0;
                d.slot = d.n_chunks = d.rot = 0;
                d.next = -1;
                dev_items[at++] = d;
            }
        }
    }
    std::vector<CombineRow> &split_rows = T.split_rows;
    split_rows.clear();
    for (size_t i = 0; i < S.items.size(); ++i) {
        const spd_work_item &w = S.items[i];
        if (w.chunk == 0 && w.n_chunks > 1)
            for (int h = 0; h < hpw_waves; ++h)  // a head-per-wave item stands for the KV heads of its group
                split_rows.push_back(CombineRow{w.slot + h * w.n_chunks, w.n_chunks, w.user, w.kv_head + h});
    }
    std::vector<RowInfo> &row_info = T.row_info;
    row_info.assign((size_t)v->n_users * Hkv, RowInfo{0, 0});
    for (const spd_work_item &w : S.items)
        if (w.chunk == 0)
            for (int h = 0; h < hpw_waves; ++h)
                row_info[(size_t)w.user * Hkv + w.kv_head + h] = RowInfo{w.slot + h * w.n_chunks, w.n_chunks};
    T.items_launched = n_groups;
    T.n_segments = (int64_t)S.items.size();
}

}  // namespace spd::host
