// Whether the buffers that one call names overlap where they must not: plain
// host arithmetic on addresses, run on every call before anything is enqueued.
// Written buffers may not overlap any other buffer, except that `out` may be
// exactly a replica of an fp32 plan (each element is read by the thread that
// writes it).  Read-only buffers may overlap each other.
//
// A call names at most four buffers besides its K replicas and K destinations,
// so these are compared with every other buffer, and destinations in ascending
// order need one pass more; only destinations in another order, or among the
// replicas' addresses, are sorted.  Sorting every call's buffers cost more host
// time than a short step's launch with many workers (measured, us per step of
// 5000 parameters in a loop, sorted / now: K=128 6.8 / 6.3, K=404 8.1 / 6.5,
// K=1000 10.8 / 7.0, with a broadcast to 1000 copies 25.8 / 11.0).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace fc {

constexpr int ALIAS_K_MAX = 1024;

struct AliasCall {
    struct Other {
        uintptr_t lo;
        bool written;
    };
    const void* const* grads = nullptr;  // K replicas of rep_bytes each, read; or null
    float* const* dst = nullptr;         // K destinations of f32_bytes each, written; or null
    int K = 0;
    uintptr_t rep_bytes = 0, f32_bytes = 0;
    Other other[4];                      // the call's other buffers, f32_bytes each
    int others = 0;
    int out = -1;                        // the one of them that may be a replica, or -1
    void add(const void* p, bool written) { other[others++] = Other{reinterpret_cast<uintptr_t>(p), written}; }
};

// Destinations against each other and against the replicas, sorted by start:
// each is compared only with the spans that start before it ends.
__attribute__((noinline)) inline bool aliased_sorted(const AliasCall& c) {
    struct Span {
        uintptr_t lo, hi;
        bool written;
    };
    Span v[2 * ALIAS_K_MAX];
    size_t n = 0;
    for (int k = 0; k < c.K; ++k) {
        const uintptr_t d = reinterpret_cast<uintptr_t>(c.dst[k]);
        v[n++] = Span{d, d + c.f32_bytes, true};
        if (c.grads) {
            const uintptr_t g = reinterpret_cast<uintptr_t>(c.grads[k]);
            v[n++] = Span{g, g + c.rep_bytes, false};
        }
    }
    std::sort(v, v + n, [](const Span& x, const Span& y) { return x.lo < y.lo; });
    for (size_t i = 0; i < n; ++i)
        for (size_t j = i + 1; j < n && v[j].lo < v[i].hi; ++j)
            if (v[i].written || v[j].written) return true;
    return false;
}

inline bool aliased(const AliasCall& c) {
    const uintptr_t R = c.rep_bytes, F = c.f32_bytes;
    if (F == 0) return false;
    auto overlap = [](uintptr_t a, uintptr_t na, uintptr_t b, uintptr_t nb) { return a < b + nb && b < a + na; };
    for (int i = 0; i < c.others; ++i)
        for (int j = i + 1; j < c.others; ++j)
            if ((c.other[i].written || c.other[j].written) && overlap(c.other[i].lo, F, c.other[j].lo, F)) return true;
    uintptr_t glo = UINTPTR_MAX, ghi = 0;  // the replicas' addresses
    if (c.grads) {
        for (int k = 0; k < c.K; ++k) {
            const uintptr_t g = reinterpret_cast<uintptr_t>(c.grads[k]);
            glo = std::min(glo, g);
            ghi = std::max(ghi, g + R);
        }
        for (int i = 0; i < c.others; ++i) {
            const uintptr_t o = c.other[i].lo;
            if (!c.other[i].written || !overlap(o, F, glo, ghi - glo)) continue;
            for (int k = 0; k < c.K; ++k) {
                const uintptr_t g = reinterpret_cast<uintptr_t>(c.grads[k]);
                if (overlap(o, F, g, R) && !(i == c.out && R == F && o == g)) return true;
            }
        }
    }
    if (c.dst) {
        bool ascending = true;
        uintptr_t dlo = UINTPTR_MAX, dhi = 0, end = 0;
        for (int k = 0; k < c.K; ++k) {
            const uintptr_t d = reinterpret_cast<uintptr_t>(c.dst[k]);
            for (int i = 0; i < c.others; ++i)
                if (overlap(c.other[i].lo, F, d, F)) return true;
            if (d < end) ascending = false;
            end = d + F;
            dlo = std::min(dlo, d);
            dhi = std::max(dhi, end);
        }
        if (!ascending || (c.grads && overlap(dlo, dhi - dlo, glo, ghi - glo))) return aliased_sorted(c);
    }
    return false;
}

}  // namespace fc
