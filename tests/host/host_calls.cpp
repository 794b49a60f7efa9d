// The library's host side on a HIP runtime that is not there: this program defines the runtime's functions itself, so that
// the built library (loaded with dlopen) allocates from the heap and every launch is recorded instead of run - only the two
// kernels that carry schedules are carried out.  Run without a GPU by tests/test_host_calls.py.
#include <dlfcn.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../include/spd.h"

struct dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string kernel;
    dim3 grid, block;
    size_t lds;
};
struct Upload {  // bytes a schedule's upload has written
    char *dst;
    size_t n;
};
static std::vector<Launch> launches;
static std::vector<Upload> uploads;

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static char *static_array()
{
    static char *p = static_cast<char *>(std::aligned_alloc(256, SPD_STATIC_SCRATCH_BYTES));
    return p;
}

static void launched(const void *fn, dim3 grid, dim3 block, void **args, size_t lds)
{
    const std::string &name = names()[fn];
    launches.push_back(Launch{name, grid, block, lds});
    const bool by_args = name.find("upload_args_kernel") != std::string::npos;
    if (by_args || name.find("upload_kernel") != std::string::npos) {
        const char *src = by_args ? static_cast<const char *>(args[0]) : *static_cast<const char **>(args[0]);
        char *dst = *static_cast<char **>(args[1]);
        const size_t n = (size_t)*static_cast<unsigned *>(args[2]) * 16;
        uploads.push_back(Upload{dst, n});
        if (!by_args || (dst >= static_array() && dst + n <= static_array() + SPD_STATIC_SCRATCH_BYTES))
            std::memcpy(dst, src, n);
    }
}

static int last_error = 0;
static bool other_capture = false;
static int this_capture = 0;

extern "C" {
struct Config {
    dim3 grid, block;
    size_t lds;
    void *stream;
};
static Config pushed;
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }  // compute units
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void **p, size_t n) { return *p = std::malloc(n), 0; }
int hipFree(void *p) { return std::free(p), 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::malloc(n), 0; }
int hipHostFree(void *p) { return std::free(p), 0; }
int hipGetSymbolAddress(void **p, const void *) { return *p = static_array(), 0; }
int hipEventCreate(void **e) { return *e = e, 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = e, 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 0.f, 0; }
int hipGetLastError()
{
    const int e = last_error;
    return last_error = 0, e;
}
// while another stream is being captured the runtime does not tell whether the null stream is: hipErrorStreamCaptureImplicit
int hipStreamIsCapturing(void *stream, int *status)
{
    if (!stream && other_capture)
        return last_error = 906;
    return *status = this_capture, 0;
}
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[fn] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    pushed = Config{grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = pushed.grid, *block = pushed.block, *lds = pushed.lds, *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, void *)
{
    launched(fn, grid, block, args, lds);
    return 0;
}
int hipExtLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, void *, void *, void *, int)
{
    launched(fn, grid, block, args, lds);
    return 0;
}
}

#define FAIL(...)                 \
    do {                          \
        std::printf(__VA_ARGS__); \
        std::printf("\n");        \
        return 1;                 \
    } while (0)

template <class F>
static F symbol(void *lib, F, const char *name)
{
    return reinterpret_cast<F>(dlsym(lib, name));
}
#define SYM(f) const auto f##_ = symbol(lib, &f, #f)

// The template arguments in a streaming kernel's mangled name (Li<value>E or, negative, Lin<value>E, and Lb<0 or 1>E).
static void template_arguments(const std::string &kernel, int32_t args[6])
{
    size_t at = kernel.find("partial_mfma_kernelI");
    if (at == std::string::npos)
        return;
    at += std::strlen("partial_mfma_kernelI");
    for (int i = 0; i < 6; ++i) {
        at += 2;  // "Li" or "Lb"
        const bool negative = kernel[at] == 'n';
        const int v = std::atoi(kernel.c_str() + at + negative);
        args[i] = negative ? -v : v;
        at = kernel.find('E', at) + 1;
    }
}

// Both owners of a step over users of `lp` and `lo` tokens; addresses are passed on, never read.
struct Step {
    spd_shape s;
    std::vector<int32_t> lens[2];
    std::vector<const void *> ptrs;
    spd_kv_view v[2] = {};
    float *buf = reinterpret_cast<float *>(0x700000000000ull);

    Step(int dtype, int Hq, int Hkv, int d, int users, int lp, int lo, bool token_major)
        : s{dtype, Hq, Hkv, d, 0.1f}, lens{std::vector<int32_t>((size_t)users, lp), std::vector<int32_t>((size_t)users, lo)}
    {
        for (int u = 0; u < users; ++u)
            ptrs.push_back(reinterpret_cast<const void *>(0x100000000ull * (uint64_t)(u + 1)));
        for (int w = 0; w < 2; ++w) {
            v[w].n_users = users;
            v[w].lens = lens[w].data();
            v[w].k_ptrs = v[w].v_ptrs = ptrs.data();
            v[w].token_stride = token_major ? (int64_t)Hkv * d : d;
            v[w].head_stride = token_major ? d : (int64_t)4096 * d;
        }
    }
};

int main(int argc, char **argv)
{
    void *lib = argc == 3 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib)
        FAIL("host_calls <library> <static LDS bytes of the whole-rows kernel>");
    SYM(spd_create);
    SYM(spd_destroy);
    SYM(spd_decode_step_static);
    SYM(spd_decode_step);
    SYM(spd_partial_attn_private);
    SYM(spd_get_schedule_stats);
    SYM(spd_get_last_kernel_instance);
    SYM(spd_set_option);
    SYM(spd_public_attn_merge);
    spd_ctx *ctx = nullptr;
    if (spd_create_(&ctx, 0) != SPD_OK)
        FAIL("spd_create");

    // the static step: each owner's schedule stays inside its own half MiB of the array.  (Its own limits say what fits; a step
    // that fits when its rows are split fits.)
    struct Case {
        int Hq, Hkv, d, users, lp, lo;
        bool token_major;
        int rc;
    };
    const Case cases[] = {
        {8, 8, 64, 2500, 64, 32, true, SPD_OK},    // an item per four heads when split, one per head when taken whole
        {16, 16, 64, 1200, 64, 32, true, SPD_OK},
        {8, 8, 64, 2000, 64, 32, true, SPD_OK},    // the largest whole-rows tables that fit: 32 bytes a row, 4 a user
        {8, 8, 64, 2016, 64, 32, true, SPD_OK},
        {8, 8, 64, 2017, 64, 32, true, SPD_OK},
        {32, 8, 128, 16, 200, 60, false, SPD_OK},
        {32, 8, 128, 2100, 40, 40, false, SPD_ERR_WORKSPACE},
    };
    constexpr size_t kHalf = 512u << 10;
    for (const Case &c : cases) {
        Step st(SPD_BF16, c.Hq, c.Hkv, c.d, c.users, c.lp, c.lo, c.token_major);
        uploads.clear();
        const int rc = spd_decode_step_static_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf, st.buf,
                                               st.buf, st.buf, st.buf, nullptr);
        if (rc != c.rc || (rc != SPD_OK && !uploads.empty()))
            FAIL("static step, %d users: %d, %zu uploads", c.users, rc, uploads.size());
        std::vector<std::pair<size_t, size_t>> at;
        for (const Upload &u : uploads) {
            const size_t b = (size_t)(u.dst - static_array()), e = b + u.n;
            if (e > 2 * kHalf || (b < kHalf && e > kHalf))
                FAIL("static step, %d users: bytes %zu..%zu leave their owner's part", c.users, b, e);
            at.push_back({b, e});
        }
        std::sort(at.begin(), at.end());
        for (size_t i = 1; i < at.size(); ++i)
            if (at[i].first < at[i - 1].second)
                FAIL("static step, %d users: the owners' tables overlap at %zu", c.users, at[i].first);
    }

    // the static step launches what spd_decode_step launches, with the same tables, wherever they fit the array: also for
    // token-major heads of 64 from 40 (32-token steps * KV heads) per unit and for groups of four of more than eight KV heads
    struct Same {
        int Hq, Hkv, d, users, lp, lo;
        bool token_major, same;
    };
    for (const Same &c : {Same{32, 8, 64, 12, 3400, 200, true, true}, Same{32, 8, 64, 12, 2900, 200, true, true},
                          Same{32, 8, 64, 9, 5000, 200, true, true}, Same{12, 12, 128, 9, 5000, 300, true, true},
                          Same{32, 32, 128, 4, 5000, 300, true, true}, Same{32, 16, 128, 20, 6000, 500, true, true},
                          Same{16, 16, 128, 40, 20000, 500, true, true}, Same{32, 8, 128, 16, 3000, 300, true, true},
                          Same{32, 8, 128, 16, 3000, 300, false, true},
                          Same{128, 8, 64, 12, 3400, 200, true, false}}) {  // its own split has partials for more than the array
        Step st(SPD_BF16, c.Hq, c.Hkv, c.d, c.users, c.lp, c.lo, c.token_major);
        std::vector<Launch> ran[2];
        for (int fixed = 0; fixed < 2; ++fixed) {
            spd_ctx *own = nullptr;
            if (spd_create_(&own, 0) != SPD_OK)
                FAIL("spd_create");
            launches.clear();
            uploads.clear();
            const int rc = (fixed ? spd_decode_step_static_ : spd_decode_step_)(own, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr,
                                                                               st.buf, st.buf, st.buf, st.buf, st.buf, st.buf, st.buf, nullptr);
            if (rc != SPD_OK)
                FAIL("%d users of %d + %d tokens, fixed %d: %d", c.users, c.lp, c.lo, fixed, rc);
            for (const Launch &l : launches)
                if (l.kernel.find("upload") == std::string::npos)
                    ran[fixed].push_back(l);
            spd_destroy_(own);
        }
        bool same = ran[0].size() == ran[1].size();
        for (size_t i = 0; same && i < ran[0].size(); ++i) {
            const Launch &a = ran[0][i], &b = ran[1][i];
            same = a.kernel == b.kernel && a.grid.x == b.grid.x && a.block.x == b.block.x && a.lds == b.lds;
        }
        if (same != c.same)
            FAIL("static step, %d users of %d + %d tokens, %d heads of %d: %s", c.users, c.lp, c.lo, c.Hkv, c.d, same ? "as the other" : "launches differ");
    }

    // calls on the null stream while another stream is being captured: new schedules, split and whole rows, and remembered ones
    other_capture = true;
    for (int again = 0; again < 2; ++again)
        for (int tokens : {5000, 90}) {
            Step st(SPD_BF16, 8, 2, 128, 1, tokens, 1, false);
            if (spd_partial_attn_private_(ctx, &st.s, st.buf, &st.v[0], st.buf, st.buf, nullptr) != SPD_OK ||
                spd_decode_step_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf, st.buf, st.buf, st.buf,
                                 st.buf, nullptr) != SPD_OK || last_error != 0)
                FAIL("%d tokens on the null stream while another stream is captured", tokens);
        }
    other_capture = false;

    // A captured step whose public rows have grown across the border between whole and split rows, while the private rows are
    // remembered split as well as whole: both owners' schedules count as found, once each, and nothing is built.
    {
        Step grown(SPD_BF16, 8, 2, 128, 1, 200, 161, false);
        auto step = [&](int pub_tokens) {
            grown.lens[1][0] = pub_tokens;
            return spd_decode_step_(ctx, &grown.s, grown.buf, &grown.v[0], &grown.v[1], nullptr, nullptr, grown.buf, grown.buf, grown.buf,
                                    grown.buf, grown.buf, grown.buf, grown.buf, nullptr);
        };
        auto whole = [] {
            bool any = false;
            for (const Launch &l : launches)
                any = any || l.kernel.find("whole_rows_kernel") != std::string::npos;
            launches.clear();
            return any;
        };
        launches.clear();
        if (step(161) != SPD_OK || !whole() || step(3001) != SPD_OK || whole())
            FAIL("which rows are taken whole");
        int64_t builds[2], hits[2];
        this_capture = 1;
        spd_get_schedule_stats_(ctx, &builds[0], &hits[0]);
        if (step(161 + 64) != SPD_OK || !whole())
            FAIL("a captured step does not keep its remembered schedules");
        spd_get_schedule_stats_(ctx, &builds[1], &hits[1]);
        this_capture = 0;
        if (builds[1] != builds[0] || hits[1] - hits[0] != 2)
            FAIL("a captured step: %lld schedules built, %lld found", (long long)(builds[1] - builds[0]), (long long)(hits[1] - hits[0]));
    }

    // The mapping of token-major calls on both sides of its lines: the KV heads (waves) of a workgroup, 0 the head-major mapping, at
    // exactly so many (32-token steps * KV heads) per unit.
    struct Mapped {
        bool fused;
        int Hq, Hkv, d, users, head_steps, below, waves;
    };
    const Mapped mapped[] = {
        // fused steps of more than eight KV heads: groups of four below 340 where four divides them, else the widest up to eight
        {true, 12, 12, 128, 16, 66, 0, 4}, {true, 12, 12, 128, 16, 340, 1, 4}, {true, 12, 12, 128, 16, 340, 0, 6},
        {true, 16, 16, 128, 16, 340, 1, 4}, {true, 16, 16, 128, 16, 340, 0, 8}, {true, 40, 20, 64, 16, 340, 1, 4}, {true, 40, 20, 64, 16, 340, 0, 5},
        {true, 28, 28, 128, 16, 340, 1, 4}, {true, 28, 28, 128, 16, 340, 0, 7}, {true, 32, 32, 128, 3, 66, 0, 4}, {true, 32, 32, 64, 16, 340, 0, 8},
        {true, 10, 10, 128, 16, 66, 0, 5}, {true, 18, 18, 128, 16, 66, 0, 6}, {true, 80, 16, 64, 1, 66, 0, 4},
        // one owner: the widest
        {false, 12, 12, 128, 16, 66, 0, 6}, {false, 16, 16, 128, 16, 66, 0, 8}, {false, 32, 32, 64, 16, 339, 0, 8},
        // up to eight KV heads: groups of four up to 900
        {true, 32, 8, 128, 16, 65, 1, 0}, {true, 32, 8, 128, 16, 65, 0, 4}, {true, 32, 8, 128, 16, 900, 1, 4}, {true, 32, 8, 128, 16, 900, 0, 8},
        {true, 24, 6, 128, 16, 65, 0, 3}, {true, 16, 4, 64, 24, 65, 1, 0}, {true, 16, 4, 64, 24, 65, 0, 4},
        // heads of 64 from 40, one owner 32; one owner's heads of 128 with up to four query heads 41; from 80 rows on
        {true, 32, 8, 64, 10, 40, 1, 0}, {true, 32, 8, 64, 10, 40, 0, 4}, {true, 32, 8, 64, 9, 64, 0, 0}, {true, 64, 16, 64, 5, 40, 0, 4},
        {false, 32, 8, 64, 10, 32, 1, 0}, {false, 32, 8, 64, 10, 32, 0, 4}, {false, 32, 8, 64, 9, 64, 0, 0},
        {false, 32, 8, 128, 10, 41, 1, 0}, {false, 32, 8, 128, 10, 41, 0, 4}, {false, 40, 8, 128, 10, 64, 0, 0}, {false, 40, 8, 128, 10, 65, 0, 4},
    };
    for (const Mapped &m : mapped) {
        const int steps = (m.head_steps * 256 + std::max(8, m.Hkv) - 1) / std::max(8, m.Hkv) - m.below - (m.fused ? m.users : 0);
        for (int form = 0; form < (m.fused ? 4 : 3); ++form) {  // bf16; fp16; in pages of 32; with the append
            Step st(form == 1 ? SPD_F16 : SPD_BF16, m.Hq, m.Hkv, m.d, m.users, steps / m.users * 32, 1, true);
            st.lens[0][0] += steps % m.users * 32 - 31;  // (the last of its steps is one token)
            for (spd_kv_view &v : st.v)
                if (form == 2) {
                    v.block_size = 32;
                    v.k_pool = v.v_pool = v.block_table = reinterpret_cast<int32_t *>(st.buf);
                    v.max_blocks = 1 << 20;
                    v.block_stride = v.block_size * v.token_stride;
                }
            const float *token = form == 3 ? st.buf : nullptr;
            spd_ctx *ctx = nullptr;
            if (spd_create_(&ctx, 0) != SPD_OK)
                FAIL("spd_create");
            launches.clear();
            const int rc = m.fused ? spd_decode_step_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], token, token, st.buf, st.buf, st.buf, st.buf,
                                                      st.buf, st.buf, st.buf, nullptr)
                                   : spd_partial_attn_private_(ctx, &st.s, st.buf, &st.v[0], st.buf, st.buf, nullptr);
            int waves = -1;
            for (const Launch &l : launches)
                if (l.kernel.find("partial_mfma_kernel") != std::string::npos) {
                    int32_t args[6];
                    template_arguments(l.kernel, args);
                    waves = args[4] ? (int)l.block.x / 64 : 0;
                }
            spd_destroy_(ctx);
            if (rc != SPD_OK || waves != m.waves)
                FAIL("mapping, fused %d, form %d, %d heads of %d, %d users, %d head steps - %d: %d, %d waves", m.fused, form, m.Hkv, m.d, m.users,
                     m.head_steps, m.below, rc, waves);
        }
    }

    // Captured calls over views that have grown across a line of the other rules: the schedules built on the near side serve them.
    // entry 0: the fused step, 1: one owner; eager at lp + lo tokens, captured 64 later (the fused step's public rows, the owner's).
    struct Line {
        int entry, Hq, Hkv, d, users, lp, lo;
        bool token_major;
        const char *what;
    };
    const Line lines[] = {
        {0, 32, 8, 64, 12, 3200, 160, true, "fused, heads of 64: 39 and 40 head steps"},
        {1, 32, 8, 64, 12, 2720, 0, true, "one owner, heads of 64: 31 and 32"},
        {1, 32, 8, 128, 12, 3488, 0, true, "one owner, heads of 128: 40 and 41"},
        {0, 32, 8, 128, 16, 4096, 32, true, "fused, heads of 128: 64 and 66"},
        {0, 16, 16, 128, 32, 5376, 32, true, "fused, groups of four and eight of sixteen heads: 338 and 342"},
        {0, 32, 8, 128, 32, 28672, 64, true, "fused, groups of four and eight of eight heads: 898 and 900"},
        {1, 32, 8, 128, 16, 8192, 0, false, "one owner, two and three pieces per unit: 64 and 65 steps"},
    };
    for (const Line &l : lines) {
        Step st(SPD_BF16, l.Hq, l.Hkv, l.d, l.users, l.lp, l.lo, l.token_major);
        spd_ctx *ctx = nullptr, *fresh = nullptr;
        if (spd_create_(&ctx, 0) != SPD_OK || spd_create_(&fresh, 0) != SPD_OK)
            FAIL("spd_create");
        auto call = [&](spd_ctx *c, std::string *ran) {
            launches.clear();
            const int rc = l.entry == 1 ? spd_partial_attn_private_(c, &st.s, st.buf, &st.v[0], st.buf, st.buf, nullptr)
                                        : spd_decode_step_(c, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf,
                                                           st.buf, st.buf, st.buf, st.buf, nullptr);
            for (const Launch &x : launches)
                if (x.kernel.find("partial_mfma_kernel") != std::string::npos)
                    *ran = x.kernel + " " + std::to_string(x.grid.x) + " x " + std::to_string(x.block.x);
            return rc;
        };
        int64_t builds[2], hits;
        std::string eager, captured, anew;
        int rc = call(ctx, &eager);
        for (int32_t &n : st.lens[l.entry == 1 ? 0 : 1])
            n += 64;
        if (rc == SPD_OK)
            rc = call(fresh, &anew);
        spd_get_schedule_stats_(ctx, &builds[0], &hits);
        this_capture = 1;
        if (rc == SPD_OK)
            rc = call(ctx, &captured);
        this_capture = 0;
        spd_get_schedule_stats_(ctx, &builds[1], &hits);
        spd_destroy_(ctx);
        spd_destroy_(fresh);
        if (rc != SPD_OK || eager == anew || captured != eager || builds[1] != builds[0])
            FAIL("capture, %s: %d, %lld built, eager %s, captured %s, anew %s", l.what, rc, (long long)(builds[1] - builds[0]), eager.c_str(),
                 captured.c_str(), anew.c_str());
    }

    // ... and over random views, options and growth, of the owners that can grow: nothing is built, each owner's schedule found once
    {
        uint32_t seed = 12345;
        auto below = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
        auto one_of = [&](std::initializer_list<int> l) { return *(l.begin() + below((int)l.size())); };
        int across = 0;
        for (int i = 0; i < 30000; ++i) {
            const int Hkv = one_of({2, 4, 6, 7, 8, 8, 9, 12, 16, 32}), G = one_of({1, 2, 4, 8, 16}), d = one_of({64, 128}), entry = below(3);
            const int users = 1 + below(one_of({2, 20, 80})), dtype = one_of({SPD_F32, SPD_BF16, SPD_F16}), top = one_of({100, 700, 3000, 9000, 30000});
            const bool token_major = below(3) != 0, even = below(4) == 0, both = below(3) == 0;
            const int grow = 1 + below(64), mapping = below(4) ? -1 : one_of({0, 1, 2, 4, 8}), round = below(6) ? 2 : one_of({1, 3, 4});
            Step st(dtype, Hkv * G, Hkv, d, users, top, top, token_major);
            if (!even)
                for (std::vector<int32_t> &lens : st.lens)
                    for (int32_t &n : lens)
                        n = 1 + below(&lens == &st.lens[1] && both ? 300 : top);
            auto call = [&](spd_ctx *c, std::string *ran) {
                launches.clear();
                const int rc = entry == 0   ? spd_decode_step_(c, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf,
                                                               st.buf, st.buf, st.buf, st.buf, nullptr)
                               : entry == 1 ? spd_partial_attn_private_(c, &st.s, st.buf, &st.v[0], st.buf, st.buf, nullptr)
                                            : spd_public_attn_merge_(c, &st.s, st.buf, &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf, st.buf,
                                                                     st.buf, st.buf, st.buf, nullptr);
                for (const Launch &x : launches)
                    if (x.kernel.find("upload") == std::string::npos)
                        *ran += x.kernel + " " + std::to_string(x.grid.x) + " x " + std::to_string(x.block.x) + "; ";
                return rc;
            };
            spd_ctx *c[2];
            std::string ran[3];
            int rc = 0;
            for (spd_ctx *&x : c)
                rc |= spd_create_(&x, 0) | spd_set_option_(x, SPD_OPT_HEAD_PER_WAVE, mapping) | spd_set_option_(x, SPD_OPT_TARGET_WG_PER_CU, round);
            rc |= call(c[0], &ran[0]);
            for (int w = 0; w < 2; ++w)
                if (entry == 0 ? w == 1 || both : w == (entry == 1 ? 0 : 1))
                    for (int32_t &n : st.lens[w])
                        n += grow;
            int64_t builds[2], hits[2];
            spd_get_schedule_stats_(c[0], &builds[0], &hits[0]);
            this_capture = 1;
            rc |= call(c[0], &ran[1]);
            this_capture = 0;
            spd_get_schedule_stats_(c[0], &builds[1], &hits[1]);
            rc |= call(c[1], &ran[2]);
            across += ran[1] != ran[2];
            for (spd_ctx *x : c)
                spd_destroy_(x);
            if (rc != SPD_OK || builds[1] != builds[0] || hits[1] - hits[0] != (entry == 0 ? 2 : 1))
                FAIL("capture, random view %d (entry %d, %d x %d heads of %d, %d users, grown by %d, options %d, %d): %d, %lld built, %s / %s", i, entry,
                     Hkv, G, d, users, grow, mapping, round, rc, (long long)(builds[1] - builds[0]), ran[0].c_str(), ran[1].c_str());
        }
        if (across < 3000)
            FAIL("capture, random views: only %d differ from a view anew", across);
    }

    // Half steps, both sides of the rule's lines (256 units: an owner's resident round is 512 pieces, 768 where it is alone): tokens per
    // user of 16 users with eight KV heads unless said otherwise.  The streaming kernel's form is its second argument's sign.
    struct Form {
        int users, lp, lo, page;
        bool one_owner, half;
        const char *what;
    };
    const Form forms[] = {
        {16, 1536, 1, 0, false, true, "12 steps a piece"},
        {16, 1504, 1, 0, false, false, "fewer"},
        {16, 3008, 736, 0, false, true, "1024 pieces, the second owner's a quarter (5.75 in 23.5 steps)"},
        {16, 3008, 768, 0, false, false, "1024 pieces, the second owner's longer"},
        {16, 3008, 3008, 0, false, false, "1024 equal pieces"},
        {16, 6000, 24000, 16, false, false, "the second owner's four times as long, in pages"},
        {16, 1536, 256, 0, false, true, "768 pieces, all resident, the second owner's a third"},
        {16, 1536, 320, 0, false, false, "896 pieces, the second owner's more than a quarter"},
        {16, 12288, 1, 16, false, true, "pages, 96 steps a piece"},
        {16, 12289, 1, 16, false, false, "pages, more"},
        {16, 12289, 1, 0, false, true, "the same rows without pages"},
        {16, 9216, 1, 16, true, true, "pages, one owner, 48 steps a piece"},
        {16, 9217, 1, 16, true, false, "pages, one owner, more"},
        {33, 3000, 1, 0, true, true, "744 segments in 512 pieces"},
        {35, 3000, 1, 0, true, false, "776 segments"},
    };
    for (const Form &f : forms) {
        Step st(SPD_BF16, 32, 8, 128, f.users, f.lp, f.lo, false);
        for (spd_kv_view &v : st.v)
            if (f.page) {
                v.block_size = f.page;
                v.k_pool = v.v_pool = v.block_table = reinterpret_cast<int32_t *>(st.buf);
                v.max_blocks = 1 << 20;
                v.head_stride = (int64_t)f.page * 128;
                v.block_stride = 8 * v.head_stride;
            }
        spd_ctx *ctx = nullptr;  // (one of its own: a view's schedule also serves the same view grown)
        if (spd_create_(&ctx, 0) != SPD_OK)
            FAIL("spd_create");
        launches.clear();
        const int rc = f.one_owner ? spd_partial_attn_private_(ctx, &st.s, st.buf, &st.v[0], st.buf, st.buf, nullptr)
                                   : spd_decode_step_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf,
                                                      st.buf, st.buf, st.buf, st.buf, nullptr);
        bool half = false, streaming = false;
        for (const Launch &l : launches) {
            streaming = streaming || l.kernel.find("partial_mfma_kernelILi1E") != std::string::npos;
            half = half || l.kernel.find("partial_mfma_kernelILi1ELin128E") != std::string::npos;
        }
        int32_t got[6] = {}, ran[6] = {};
        spd_get_last_kernel_instance_(ctx, got);
        for (const Launch &l : launches)
            template_arguments(l.kernel, ran);
        if (std::memcmp(got, ran, sizeof got) != 0)
            FAIL("%s: the last instance is not what ran: <%d, %d, ..>, <%d, %d, ..>", f.what, got[0], got[1], ran[0], ran[1]);
        spd_destroy_(ctx);
        if (rc != SPD_OK || !streaming || half != f.half)
            FAIL("half steps, %d users of %d + %d tokens (%s): %d, %d", f.users, f.lp, f.lo, f.what, rc, half);
    }

    // fp32 rows through descriptors (the negative second argument of dtype 3): contiguous, end to end and without an append
    struct Fp32 {
        int users, stride;
        bool token_major, append, range;
    };
    for (const Fp32 &f : {Fp32{16, 128, false, false, true}, Fp32{48, 128, false, false, true}, Fp32{16, 128, false, true, false},
                          Fp32{16, 1024, true, false, false}, Fp32{16, 132, false, false, false}}) {
        Step st(SPD_F32, 32, 8, 128, f.users, 3000, 3000, f.token_major);
        for (spd_kv_view &v : st.v)
            v.token_stride = f.stride;
        spd_ctx *ctx = nullptr;
        if (spd_create_(&ctx, 0) != SPD_OK)
            FAIL("spd_create");
        launches.clear();
        const float *token = f.append ? st.buf : nullptr;
        const int rc = spd_decode_step_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], token, token, st.buf, st.buf, st.buf, st.buf, st.buf,
                                        st.buf, st.buf, nullptr);
        bool range = false, plain = false;
        for (const Launch &l : launches) {
            range = range || l.kernel.find("partial_mfma_kernelILi3ELin128E") != std::string::npos;
            plain = plain || l.kernel.find("partial_mfma_kernelILi3ELi128E") != std::string::npos;
        }
        int32_t got[6] = {}, ran[6] = {};
        spd_get_last_kernel_instance_(ctx, got);
        for (const Launch &l : launches)
            template_arguments(l.kernel, ran);
        if (std::memcmp(got, ran, sizeof got) != 0)
            FAIL("fp32 rows: the last instance is not what ran: <%d, %d, ..>, <%d, %d, ..>", got[0], got[1], ran[0], ran[1]);
        spd_destroy_(ctx);
        if (rc != SPD_OK || range != f.range || plain == range)
            FAIL("fp32 rows, %d users, stride %d: %d, %d, %d", f.users, f.stride, rc, range, plain);
    }

    // whole rows: no launch asks for more than 64 KB of LDS, the kernel's static part (argv[2], from the compiler's report) and
    // the slots together
    const size_t static_lds = (size_t)std::atoi(argv[2]);
    for (int G = 1; G <= 16; ++G)
        for (int d = 64; d <= 128; d *= 2)
            for (int dtype : {SPD_F32, SPD_BF16, SPD_F16}) {
                const int tile = dtype == SPD_F32 && d == 128 ? 16 : 32;
                for (int steps = 1; steps <= 12; ++steps) {
                    Step st(dtype, 2 * G, 2, d, 1, steps * tile, 1, false);
                    launches.clear();
                    if (spd_decode_step_(ctx, &st.s, st.buf, &st.v[0], &st.v[1], nullptr, nullptr, st.buf, st.buf, st.buf, st.buf, st.buf,
                                         st.buf, st.buf, nullptr) != SPD_OK)
                        FAIL("step");
                    const Launch &l = launches.back();
                    if (l.kernel.find("whole_rows_kernel") == std::string::npos)
                        FAIL("G = %d, %d steps: %s", G, steps, l.kernel.c_str());
                    const size_t slots = l.lds / (l.block.x / 64 + 1), need = (size_t)G * d * sizeof(float);
                    if (l.block.x > 768 || slots < need || l.lds + static_lds > 64 * 1024)
                        FAIL("G = %d, d = %d, %u threads: %zu + %zu bytes of LDS", G, d, l.block.x, l.lds, static_lds);
                }
            }
    spd_destroy_(ctx);
    std::printf("ok\n");
    std::fflush(stdout);
    _Exit(0);
}
