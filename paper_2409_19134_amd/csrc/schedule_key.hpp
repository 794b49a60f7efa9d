// The key a schedule is remembered by: the bytes of a view that determine its split schedule (host only, no HIP calls).
#pragma once
#include <cstdint>
#include <cstring>
#include <vector>

#include "../../include/spd.h"

namespace spd::host {

// Hash of a schedule key (keys grow with the number of users and are hashed on every call): four chains of eight bytes each, which
// the processor runs side by side.  Only a filter: a hit is confirmed by comparing the keys themselves.
inline uint64_t hash_key(const uint8_t *p, size_t n)
{
    constexpr uint64_t mul = 0x9E3779B97F4A7C15ull;
    uint64_t h = 1469598103934665603ull ^ n, c[4] = {h, h + 1, h + 2, h + 3};
    size_t i = 0;
    auto word = [p](size_t at) {
        uint64_t w;
        std::memcpy(&w, p + at, 8);
        return w;
    };
    for (; i + 32 <= n; i += 32)
        for (size_t k = 0; k < 4; ++k) {
            c[k] = (c[k] ^ word(i + 8 * k)) * mul;
            c[k] ^= c[k] >> 29;
        }
    for (size_t k = 0; k < 4; ++k) {
        h = (h ^ c[k]) * mul;
        h ^= h >> 29;
    }
    for (; i + 8 <= n; i += 8) {
        h = (h ^ word(i)) * mul;
        h ^= h >> 29;
    }
    for (; i < n; ++i)
        h = (h ^ p[i]) * 1099511628211ull;
    return h;
}

// A decode loop appends one token per user and step: a schedule built for the lengths L serves L + g for
// 1 <= g <= kMaxGrow as well (the kernels add g to the end of every row's last segment), which spares the loop a
// rebuild and an upload per step.  Beyond that the pieces would drift out of balance and a new schedule is built.
constexpr int32_t kMaxGrow = 64;
constexpr size_t kKeyLensOffset = 6 * sizeof(int32_t);  // the lengths follow the key's six-integer head

inline uint64_t hash_key_but_lens(const std::vector<uint8_t> &key, int n_users)
{
    const size_t tail = kKeyLensOffset + sizeof(int32_t) * (size_t)n_users;
    return hash_key(key.data(), kKeyLensOffset) ^ (hash_key(key.data() + tail, key.size() - tail) * 0x9E3779B97F4A7C15ull);
}

// g if `key` is `old_key` with every length g larger (1 <= g <= kMaxGrow), else 0.
inline int32_t uniform_growth(const std::vector<uint8_t> &old_key, const std::vector<uint8_t> &key, int n_users)
{
    if (n_users == 0 || old_key.size() != key.size())
        return 0;
    const size_t tail = kKeyLensOffset + sizeof(int32_t) * (size_t)n_users;
    if (std::memcmp(old_key.data(), key.data(), kKeyLensOffset) != 0 ||
        std::memcmp(old_key.data() + tail, key.data() + tail, key.size() - tail) != 0)
        return 0;
    int32_t g = 0;
    for (int u = 0; u < n_users; ++u) {
        int32_t was, now;
        std::memcpy(&was, old_key.data() + kKeyLensOffset + sizeof(int32_t) * (size_t)u, sizeof was);
        std::memcpy(&now, key.data() + kKeyLensOffset + sizeof(int32_t) * (size_t)u, sizeof now);
        if (u == 0)
            g = now - was;
        if (now - was != g || g < 1 || g > kMaxGrow)
            return 0;
    }
    return g;
}

// tuning: the kTuningInts integers of the context's Tuning (they shape the schedule like the lengths do).  Made anew on every call, so
// written in place, without an insertion per item (host work of a fused step over 256 users, this, the hash and one validation
// instead of two: 13.0 -> 2.5 us; 32 users 1.8 -> 0.4).
inline void make_key(const spd_shape *s, const spd_kv_view *v, int hpw, const int32_t *tuning, int n_tuning,
                     std::vector<uint8_t> &key)
{
    // the items carry row base addresses (contiguous mode) or row offsets inside the pools (paged mode): the key holds
    // everything those depend on.  The pools themselves are not part of it, so the layers of a model, which share
    // lengths and block table but have a pool each, share one schedule.
    const size_t users = (size_t)v->n_users;
    const int32_t tables = (v->block_size == 0 && v->k_ptrs_dev) ? 1 : 0;  // the items then hold offsets, not addresses
    const bool strides = v->head_strides && v->block_size == 0, pointers = v->block_size == 0 && !tables;
    const int32_t head[6] = {s->dtype, s->n_q_heads, s->n_kv_heads, v->n_users, v->block_size,
                             hpw};
    static_assert(sizeof head == kKeyLensOffset, "the lengths follow the head");
    const size_t size = sizeof head + users * sizeof(int32_t) + sizeof tables + (size_t)n_tuning * sizeof(int32_t) + sizeof v->head_stride +
                        (strides ? users * sizeof(int64_t) : 0) + (pointers ? users * 2 * sizeof(void *) : 0);
    if (key.size() != size)  // (the same view on the next call: written over in place)
        key.resize(size);
    uint8_t *at = key.data();
    auto put = [&at](const void *p, size_t n) {
        if (n)
            std::memcpy(at, p, n);
        at += n;
    };
    put(head, sizeof head);
    put(v->lens, users * sizeof(int32_t));
    put(&tables, sizeof tables);
    put(tuning, sizeof(int32_t) * (size_t)n_tuning);
    put(&v->head_stride, sizeof v->head_stride);
    if (strides)
        put(v->head_strides, users * sizeof(int64_t));
    if (pointers)
        for (size_t u = 0; u < users; ++u) {  // pointers of empty users are never read: normalise them
            const void *kv[2] = {v->lens[u] ? v->k_ptrs[u] : nullptr, v->lens[u] ? v->v_ptrs[u] : nullptr};
            put(kv, sizeof kv);
        }
}

}  // namespace spd::host
