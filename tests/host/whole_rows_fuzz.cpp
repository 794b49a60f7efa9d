// Host-only fuzz driver for the whole-rows tables and the rule that picks them, against the split schedule's tables for the
// same view.  Built by tests/test_whole_rows_host.py with AddressSanitizer and UBSan, run without a GPU.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_2409_19134_amd/csrc/schedule.hpp"

using namespace spd::host;

static uint64_t state = 0x9e3779b97f4a7c15ull;
static uint64_t rnd()
{
    state ^= state << 7;
    state ^= state >> 9;
    return state * 0x2545f4914f6cdd1dull;
}

#define FAIL(...)                 \
    do {                          \
        std::printf(__VA_ARGS__); \
        std::printf("\n");        \
        return 1;                 \
    } while (0)

// Equal rows on 256 compute units, 16-bit rows of 128 channels and 8 KV heads: on which side of the rule's lines they are.
static int measured_shapes()
{
    struct Shape {
        int users, tokens;
        bool token_major, whole;
    };
    const Shape shapes[] = {
        {1, 500, false, true}, {1, 800, false, false},      // a few rows: the excess of the longest
        {16, 500, false, true}, {16, 900, false, false},    // a row for every second unit
        {42, 1000, false, false}, {62, 1136, false, true},  // two rounds of eight waves: the second half empty, or nearly full
        {70, 900, false, false}, {81, 620, false, true},    // one round of four waves
        {107, 1755, false, false}, {105, 487, false, true}, {250, 1000, false, true},  // several: a last round of long rows
        {104, 796, true, false}, {86, 366, true, true}, {250, 800, true, true},        // what the head-per-wave mapping reads better
        {250, 2100, false, false},
    };
    for (const Shape &x : shapes) {
        std::vector<int32_t> lens((size_t)x.users, x.tokens);
        WholeRowsLoad c;
        c.Hkv = 8;
        c.n_cus = 256;
        c.n_users = x.users;
        c.lens0 = lens.data();
        if ((whole_rows_choice(c, [&](int64_t) { return x.token_major; }) != 0) != x.whole)
            FAIL("%d users of %d tokens", x.users, x.tokens);
    }
    return 0;
}

int main()
{
    if (measured_shapes())
        return 1;
    for (int iter = 0; iter < 600; ++iter) {
        const int n = (int)(rnd() % 40), Hkv = 1 + (int)(rnd() % 16), es = rnd() % 2 ? 2 : 4, d = rnd() % 2 ? 64 : 128;
        const int top = 1 + (int)(rnd() % 3000);
        std::vector<int32_t> lens((size_t)n), lens1((size_t)n);
        for (int u = 0; u < n; ++u) {
            lens[(size_t)u] = rnd() % 4 ? (int32_t)(rnd() % top) : 0;
            lens1[(size_t)u] = rnd() % 4 ? (int32_t)(rnd() % top) : 0;
        }
        // addresses are only computed, never read
        std::vector<const void *> kp((size_t)n), vp((size_t)n);
        std::vector<int64_t> strides((size_t)n);
        for (int u = 0; u < n; ++u) {
            kp[(size_t)u] = reinterpret_cast<const void *>((uintptr_t)0x100000000ull * (uintptr_t)(2 * u + 1));
            vp[(size_t)u] = reinterpret_cast<const void *>((uintptr_t)0x100000000ull * (uintptr_t)(2 * u + 2));
            strides[(size_t)u] = (int64_t)(lens[(size_t)u] + (int)(rnd() % 9)) * d;
        }
        spd_kv_view v = {};
        v.n_users = n;
        v.lens = lens.data();
        v.k_ptrs = kp.data();
        v.v_ptrs = vp.data();
        v.token_stride = d;
        v.head_stride = (int64_t)top * d;
        switch (rnd() % 4) {
        case 0: v.block_size = 16; break;                                                     // offsets in the pools
        case 1: v.head_strides = strides.data(); break;
        case 2: v.k_ptrs_dev = kp.data(), v.v_ptrs_dev = vp.data(); break;                    // offsets from the users' pointers
        default: break;
        }

        std::vector<spd::RowItem> rows;
        std::vector<int32_t> order;
        build_whole_rows(Hkv, es, &v, rows, order);
        if (rows.size() != (size_t)n * Hkv || order.size() != (size_t)n)
            FAIL("sizes");
        // the same addresses as the split schedule's items, and every token of every row
        Schedule S;
        build_schedule(Hkv, n, lens.data(), 256, 0, Tuning(), S);
        DeviceTables T;
        build_device_tables(S, Hkv, es, &v, 0, T);
        std::vector<int64_t> tokens((size_t)n * Hkv, 0);
        for (const spd::DevItem &it : T.items) {
            if (it.n_chunks == 0)
                continue;
            const spd::RowItem &r = rows[(size_t)it.user * Hkv + it.kv_head];
            if (r.k_base != it.k_base || r.v_base != it.v_base)
                FAIL("row address of user %d head %d", it.user, it.kv_head);
            tokens[(size_t)it.user * Hkv + it.kv_head] += it.t_end - it.t_begin;
        }
        for (int u = 0; u < n; ++u)
            for (int h = 0; h < Hkv; ++h)
                if (rows[(size_t)u * Hkv + h].t_end != lens[(size_t)u] || tokens[(size_t)u * Hkv + h] != lens[(size_t)u])
                    FAIL("tokens of user %d", u);
        std::vector<int32_t> seen(order);
        std::sort(seen.begin(), seen.end());
        for (int u = 0; u < n; ++u)
            if (seen[(size_t)u] != u || (u && lens[(size_t)order[(size_t)u - 1]] < lens[(size_t)order[(size_t)u]]))
                FAIL("launch order");

        // the rule: a wave count the kernel can be launched with, and the limits it promises
        WholeRowsLoad c;
        c.tile = es * d == 512 ? 16 : 32;
        c.step_bytes = 2 * c.tile * es * d;
        c.Hkv = Hkv;
        c.n_cus = 1 + (int)(rnd() % 300);
        c.n_users = n;
        c.lens0 = lens.data();
        c.lens1 = rnd() % 2 ? lens1.data() : nullptr;
        int64_t longest = 0;
        for (int u = 0; u < n; ++u)
            longest = std::max<int64_t>(longest, (lens[(size_t)u] + c.tile - 1) / c.tile +
                                                     (c.lens1 ? (lens1[(size_t)u] + c.tile - 1) / c.tile : 0));
        const bool token_major = rnd() % 2;
        auto head_per_wave = [token_major](int64_t steps) { return token_major && steps > 500; };
        const int waves = whole_rows_choice(c, head_per_wave);
        if (waves < 0 || waves > spd::kRowsMaxWaves || (waves > 1 && waves > longest))
            FAIL("%d waves for rows of up to %lld steps", waves, (long long)longest);
        if (waves > 0 && longest * c.step_bytes > kWholeRowsLimit * 16384)
            FAIL("whole rows of %lld steps", (long long)longest);
        if (longest * c.step_bytes <= kWholeRowsShort * 16384 && waves == 0)
            FAIL("rows of %lld steps are short whatever their number", (long long)longest);
        // result channels ask for up to four waves, whatever the steps
        WholeRowsLoad h = c;
        h.head_channels = 64 * (1 + (int)(rnd() % 32));
        const int least = std::min(4, (h.head_channels + 255) / 256);
        if (whole_rows_choice(h, head_per_wave) != (waves ? std::max(waves, least) : 0))
            FAIL("%d waves for %d result channels", whole_rows_choice(h, head_per_wave), h.head_channels);
        // by length as soon as a row has to wait for another's end: a unit holds three workgroups of four waves, one of eight
        for (int w : {4, 8, 12}) {
            const int64_t resident = (int64_t)c.n_cus * (w == 4 ? 3 : 1);
            if (whole_rows_by_length(resident, w, c.n_cus) || !whole_rows_by_length(resident + 1, w, c.n_cus))
                FAIL("launch order of %lld rows of %d waves", (long long)resident, w);
        }
        // the kernel's division by the wave count: x * ceil(2^32 / waves) >> 32, for every product it forms
        for (int w = 1; w <= spd::kRowsMaxWaves; ++w) {
            const uint32_t mul = (uint32_t)(((1ull << 32) + w - 1) / w);
            const uint32_t x = (uint32_t)(rnd() % (128 * spd::kRowsMaxWaves + 1));
            if (w > 1 && (uint32_t)(((uint64_t)x * mul) >> 32) != x / w)
                FAIL("%u / %d", x, w);
        }
    }
    std::printf("ok 600\n");
    return 0;
}
