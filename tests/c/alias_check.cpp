// CPU check of the overlap check (csrc/fc_alias.h), built with AddressSanitizer
// and UndefinedBehaviorSanitizer by tests/test_alias_cpu.py: random placements
// of replicas, destinations and up to four other buffers (in order, permuted,
// interleaved, touching, repeated, an output exactly on a replica), each
// verdict compared with the rule applied to every pair.
#include <cstdio>
#include <random>
#include <vector>

#include "fc_alias.h"

struct Span {
    uintptr_t lo, hi;
    bool written, replica, out;
};

static bool by_pairs(const std::vector<Span>& v, bool f32) {
    for (size_t i = 0; i < v.size(); ++i)
        for (size_t j = i + 1; j < v.size(); ++j) {
            const Span &a = v[i], &b = v[j];
            if (a.lo == a.hi || b.lo == b.hi || !(a.lo < b.hi && b.lo < a.hi) || (!a.written && !b.written)) continue;
            if (f32 && ((a.out && b.replica) || (b.out && a.replica)) && a.lo == b.lo && a.hi == b.hi) continue;
            return true;
        }
    return false;
}

int main() {
    std::mt19937 rng(3);
    auto pick = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    long yes = 0, no = 0;
    for (int it = 0; it < 200000; ++it) {
        const int K = it % 997 == 0 ? 1024 : 1 + pick(9);
        const bool f32 = pick(2);
        const uintptr_t extent = pick(20) ? 16 * (1 + pick(3)) : 0;
        fc::AliasCall c;
        c.K = K;
        c.rep_bytes = extent * (f32 ? 4 : 2);
        c.f32_bytes = extent * 4;
        // rows of one slab, a slab in another order, or anywhere in a small arena
        const uintptr_t unit = extent * 4 + 16 * pick(2);
        auto rows = [&](uintptr_t base, bool shuffle) {
            std::vector<uintptr_t> r;
            for (int k = 0; k < K; ++k) r.push_back(base + k * unit);
            if (shuffle) std::shuffle(r.begin(), r.end(), rng);
            for (int k = 0; k < K; ++k)
                if (pick(60 * K) == 0) r[k] = 4096 + 16 * pick(8 * K);
            return r;
        };
        const uintptr_t slab = K * unit;
        const int layout = pick(4);
        const std::vector<uintptr_t> g = rows(4096, pick(3) == 0);
        std::vector<uintptr_t> d = rows(layout ? 4096 + slab + 16 * pick(3) : 4096 + 16 * pick(3), pick(3) == 0);
        if (layout == 3)  // destinations between the replicas
            for (int k = 0; k < K; ++k) d[k] = g[k] + (pick(2) ? c.rep_bytes : unit);
        std::vector<const void*> gp;
        std::vector<float*> dp;
        for (int k = 0; k < K; ++k) {
            gp.push_back(reinterpret_cast<const void*>(g[k]));
            dp.push_back(reinterpret_cast<float*>(d[k]));
        }
        std::vector<Span> all;
        if (pick(8)) {
            c.grads = gp.data();
            for (uintptr_t x : g) all.push_back(Span{x, x + c.rep_bytes, false, true, false});
        }
        if (pick(2)) {
            c.dst = dp.data();
            for (uintptr_t x : d) all.push_back(Span{x, x + c.f32_bytes, true, false, false});
        }
        const int n = pick(5);
        for (int i = 0; i < n; ++i) {
            uintptr_t x = 4096 + 2 * slab + 64 + i * unit;
            if (pick(6) == 0) x = 4096 + 16 * pick(static_cast<int>(slab / 8) + 1);
            if (pick(6) == 0) x = g[pick(K)];
            const bool written = pick(4) != 0, out = written && c.out < 0 && pick(3) == 0;
            if (out) c.out = c.others;
            c.add(reinterpret_cast<const void*>(x), written);
            all.push_back(Span{x, x + c.f32_bytes, written, false, out});
        }
        const bool want = by_pairs(all, f32), got = fc::aliased(c);
        (want ? yes : no) += 1;
        if (want != got) {
            std::fprintf(stderr, "case %d: K=%d extent %zu: %d for %d\n", it, K, (size_t)extent, got, want);
            return 1;
        }
    }
    if (yes < 10000 || no < 10000) return 2;
    std::printf("all verdicts agree (%ld overlap, %ld do not)\n", yes, no);
    return 0;
}
