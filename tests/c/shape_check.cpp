// CPU check of the split kernel's rule (csrc/fc_shape.h, default_split) and of
// the association it leads to, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_shape_cpu.py.  For every worker
// count and many plan widths it checks what the kernel relies on -- waves,
// runs, LDS and stack within their limits, a thread per element, batches of
// pointers inside the padded table -- and that the sums of runs, batch by
// batch and then wave by wave, give the bits of the tree over all replicas.
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "fc_shape.h"

static int failures = 0;
#define CHECK(c, ...)                                   \
    do {                                                \
        if (!(c)) {                                     \
            if (failures++ < 20) {                      \
                std::fprintf(stderr, __VA_ARGS__);      \
                std::fprintf(stderr, " [%s]\n", #c);    \
            }                                           \
        }                                               \
    } while (0)

// neighbours paired level by level, an odd last one moving up unchanged
static float tree(std::vector<float> x) {
    while (x.size() > 1) {
        std::vector<float> y;
        for (size_t i = 0; i < x.size(); i += 2) y.push_back(i + 1 < x.size() ? x[i] + x[i + 1] : x[i]);
        x = y;
    }
    return x[0];
}

// one wave's run: whole batches of 16 on a binary counter, the rest first
static float run_sum(const float* p, int n) {
    std::vector<float> st;
    std::vector<int> size;
    const int full = n / 16;
    for (int c = 0; c < full; ++c) {
        float s = tree(std::vector<float>(p + 16 * c, p + 16 * c + 16));
        int k = 1;
        while (!size.empty() && size.back() == k) {
            s = st.back() + s;
            k += size.back();
            st.pop_back();
            size.pop_back();
        }
        st.push_back(s);
        size.push_back(k);
    }
    CHECK(st.size() <= 3 && full < 8, "stack %zu of %d replicas", st.size(), n);
    bool have = n % 16;
    float acc = have ? tree(std::vector<float>(p + 16 * full, p + n)) : 0.0f;
    while (!st.empty()) {
        acc = have ? st.back() + acc : st.back();
        have = true;
        st.pop_back();
    }
    return acc;
}

int main() {
    std::mt19937 rng(7);
    std::normal_distribution<float> gauss;
    const int cus = 256;
    long plans = 0;
    for (int K = 1; K <= 1024; ++K) {
        std::vector<float> x(K);
        for (float& v : x) v = gauss(rng);
        const float want = tree(x);
        for (uint64_t n64 : {1, 2, 65, 130, 255, 256, 511, 512, 513, 1024, 1500, 2048, 3000, 4096, 6144, 6145, 90000}) {
            for (int f16 = 0; f16 < 2; ++f16) {
                for (int is_tree = 0; is_tree < 2; ++is_tree) {
                    fc::Shape sh{};
                    const uint64_t n128 = (n64 + 1) / 2, n256 = (n64 + 3) / 4;
                    if (!fc::default_split(f16 ? FC_F16 : FC_F32, is_tree, K, cus, 160 << 10, n256, n128, n64, sh)) {
                        CHECK(sh.lane == 0, "lane without the kernel");
                        continue;
                    }
                    ++plans;
                    CHECK(K > 16 && n256 <= 6 * cus, "K=%d tiles %llu", K, (unsigned long long)n256);
                    CHECK(sh.lane == 1 || sh.lane == 2, "lane %d", sh.lane);
                    CHECK(sh.waves >= sh.lane && sh.waves <= fc::SPLIT_WAVES, "K=%d waves %d", K, sh.waves);
                    CHECK(sh.block == 64 * sh.waves, "block %d", sh.block);
                    if (is_tree) {
                        CHECK(sh.run == 16 || sh.run == 32 || sh.run == 64, "run %d", sh.run);
                        CHECK((sh.waves - 1) * sh.run < K && K <= sh.waves * sh.run, "K=%d %d x %d", K, sh.waves, sh.run);
                        std::vector<float> sums;
                        for (int q = 0; q < sh.waves; ++q)
                            sums.push_back(run_sum(&x[q * sh.run], std::min(sh.run, K - q * sh.run)));
                        const float got = tree(sums);
                        CHECK(std::memcmp(&got, &want, 4) == 0, "K=%d run %d: %a for %a", K, sh.run, got, want);
                    } else if (sh.chain) {
                        CHECK(sh.lane == 1 && sh.waves >= 2 && n64 <= (uint64_t)cus, "chain of %d waves", sh.waves);
                        CHECK(2 * (sh.waves - 1) * 16 * 64 * 4 <= fc::CHAIN_LDS && fc::CHAIN_LDS <= 160 << 10, "LDS");
                    } else {
                        CHECK(sizeof(float) * 64 * sh.lane * sh.waves * 16 <= 65536, "LDS of %d x %d", sh.lane, sh.waves);
                        CHECK((sh.waves - 1) * 16 < K || sh.waves == sh.lane, "K=%d waves %d", K, sh.waves);
                    }
                    // the last batch starts at a replica: its pointers end inside the pad
                    CHECK((K - 1) / 16 * 16 + 15 < K + fc::TABLE_PAD, "pad for K=%d", K);
                }
            }
        }
    }
    if (failures) return 1;
    std::printf("all shapes valid (%ld plans)\n", plans);
    return 0;
}
