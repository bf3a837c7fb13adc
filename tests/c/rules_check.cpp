// CPU check of the rules by which calls choose their launches (csrc/fc_shape.h),
// run by tests/test_rules_cpu.py: `rules_check NAME` checks one rule at the sizes
// where it was measured and over its range.
#include <cstdio>
#include <cstring>

#include "fc_shape.h"

static int failures = 0;
#define CHECK(c, ...)                                \
    do {                                             \
        if (!(c)) {                                  \
            if (failures++ < 20) {                   \
                std::fprintf(stderr, __VA_ARGS__);   \
                std::fprintf(stderr, " [%s]\n", #c); \
            }                                        \
        }                                            \
    } while (0)

static fc::Shape shape(int block, int vecs, int lane = 0) {
    fc::Shape sh{};
    sh.block = block;
    sh.vecs = vecs;
    sh.lane = lane;
    return sh;
}

// blocks that share a broadcast tile's destinations
static void copies() {
    const fc::Shape u4 = shape(256, 4), one = shape(64, 1), split = shape(512, 1, 1);
    auto tiles = [](uint64_t n, uint64_t per) { return static_cast<int>((n + per - 1) / per); };
    for (int K = 1; K <= 1024; ++K)
        for (uint64_t n : {1000ull, 65536ull, 131072ull, 262144ull, 300000ull, 600000ull, 1000000ull, 3000000ull})
            for (const fc::Shape& sh : {u4, one, split}) {
                const int grid = tiles(n, sh.lane ? 64 * sh.lane : sh.block * sh.vecs * 4);
                const int g = fc::bcast_groups(sh, K, grid, n, 0);
                CHECK(g >= 1 && g <= (K + 7) / 8, "K=%d n=%llu: %d", K, (unsigned long long)n, g);
                // a caller's cap holds, also where it is wider than the grid
                for (int cap : {grid, grid + 1, 3 * grid, 100 * grid}) {
                    const int c = fc::bcast_groups(sh, K, grid, n, cap);
                    CHECK(c >= 1 && c <= g && c * grid <= cap, "K=%d cap %d: %d x %d", K, cap, c, grid);
                }
                // writes bound the copies of larger plans
                CHECK(n <= 262144 || g == 1, "K=%d n=%llu: %d", K, (unsigned long long)n, g);
            }
    CHECK(fc::bcast_groups(one, 1000, tiles(4000, 256), 4000, 0) == 125, "4000 x K=1000");
    CHECK(fc::bcast_groups(u4, 64, tiles(262144, 4096), 262144, 0) == 8, "262144 x K=64");
    CHECK(fc::bcast_groups(one, 200, tiles(100000, 256), 100000, 0) == 1, "100000 x K=200");
}

// resident broadcasts that pack their tiles' descriptors
static void packed() {
    CHECK(fc::bcast_packed(8, 214 * 256, 256, 0), "213 tiles a block");
    CHECK(!fc::bcast_packed(8, 32 * 256, 256, 0) && fc::bcast_packed(8, 32 * 256 + 1, 256, 0), "two tiles a wave");
    CHECK(!fc::bcast_packed(3, 214 * 256, 256, 0), "few destinations");
    CHECK(!fc::bcast_packed(128, 4096, 64, 64), "capped grid");
}

static void expect(const fc::Shape& sh, int vecs, int kchunk, int block, const char* what) {
    CHECK(sh.vecs == vecs && sh.kchunk == kchunk && sh.block == block, "%s: (%d, %d, %d)", what, sh.vecs, sh.kchunk,
          sh.block);
}

// shapes of plans with an explicit schedule or a capped grid
static void shapes() {
    for (int c = 0; c < 4; ++c)
        for (int K = 1; K <= 1024; ++K) {
            const uint64_t n = (uint64_t(1) << 23) - c % 2;
            const bool capped = c >= 2, few = c > 0;
            fc::Shape sh{};
            fc::default_shape(FC_F16, K, n, capped, sh);
            expect(sh, 4, 4, 256, "fp16");
            fc::default_shape(FC_F32, K, n, capped, sh);
            if (K <= 2 || (few && K <= 4)) expect(sh, 1, 8, 256, "few replicas");
            else if (K > 16 && K <= 64) expect(sh, 4, 2, 256, "17 to 64 replicas");
            else expect(sh, 1, 16, 64, "other");
        }
}

// shapes of default plans' short steps that one wave per tile serves
static void short_steps() {
    auto of = [](fc_dtype t, int K, uint64_t n) {
        fc::Shape sh{};
        fc::short_shape(t, K, 256, (n + 255) / 256, (n + 1023) / 1024, sh);
        return sh;
    };
    for (uint64_t n : {64ull, 8000ull, 262144ull, 300000ull, 520000ull, 800000ull, 1048576ull})
        for (int K = 1; K <= 16; ++K) {
            if (K <= 4) expect(of(FC_F32, K, n), 1, 8, 256, "fp32, one batch half empty");
            if (K > 8) expect(of(FC_F32, K, n), 1, 16, 64, "fp32, one batch of 16");
            if (K > 4) expect(of(FC_F16, K, n), 1, 16, 64, "fp16");
        }
    for (uint64_t n : {53568ull, 262144ull, 520000ull, 1048576ull, 1115480ull})
        expect(of(FC_F32, 8, n), 1, 8, 256, "fp32 K=8, rounds filled");
    for (uint64_t n : {300000ull, 400000ull, 800000ull}) expect(of(FC_F32, 8, n), 1, 16, 64, "fp32 K=8, last round empty");
    for (int K = 1; K <= 4; ++K) {
        expect(of(FC_F16, K, 1000), 4, 4, 256, "fp16, one block");
        expect(of(FC_F16, K, 800000), 4, 4, 256, "fp16, many tiles");
        if (K <= 2) expect(of(FC_F16, K, 100000), 1, 8, 256, "fp16 K <= 2");
        else expect(of(FC_F16, K, 100000), 1, 16, 64, "fp16 K = 3, 4");
    }
    expect(of(FC_F32, 32, 300000), 1, 16, 64, "fp32 K=32, last round empty");
    expect(of(FC_F32, 32, 460000), 1, 8, 256, "fp32 K=32, rounds filled");
}

// the plans that the split kernel serves
static void split_plans() {
    auto is = [](fc_dtype t, bool tree, int K, uint64_t n) {
        fc::Shape sh{};
        return fc::default_split(t, tree, K, 256, 160 << 10, (n + 255) / 256, (n + 127) / 128, (n + 63) / 64, sh);
    };
    for (fc_dtype t : {FC_F32, FC_F16})
        for (int K : {33, 64, 128, 200, 399, 400, 512, 1024}) {
            const bool many = t == FC_F32 && K >= 400;
            CHECK(is(t, true, K, 196608), "tree K=%d, 3 tiles per unit", K);
            CHECK(is(t, true, K, 262144) == !many, "tree K=%d, 4 tiles per unit", K);
            CHECK(!is(t, true, K, 262145) && !is(t, true, K, 300000) && !is(t, true, K, 393216), "tree K=%d", K);
            CHECK(is(t, false, K, 262144), "linear K=%d, 4 tiles per unit", K);
            CHECK(is(t, false, K, 300000) == (t == FC_F32), "linear K=%d, 4.6 tiles per unit", K);
            CHECK(!is(t, false, K, 393216), "linear K=%d, 6 tiles per unit", K);
        }
    CHECK(is(FC_F16, true, 128, 163696) && is(FC_F32, false, 1000, 10304), "short plans of many workers");
    CHECK(!is(FC_F32, true, 16, 4096) && !is(FC_F32, true, 32, 131072) && is(FC_F32, true, 32, 130000), "K <= 32");
}

// allocation-free steps that run in two passes
static void noalloc() {
    for (int K = 1; K <= 1024; ++K)
        for (int bytes : {2, 4}) {
            CHECK(fc::noalloc_two_pass(FC_SCHED_FUSED, false, K, bytes, 100, 0) == (K * bytes > 256), "fused K=%d", K);
            CHECK(fc::noalloc_two_pass(FC_SCHED_TWO_PASS, false, K, bytes, 100, 0), "two passes K=%d", K);
            CHECK(!fc::noalloc_two_pass(FC_SCHED_TWO_PASS, true, K, bytes, 100, 0), "passes joined K=%d", K);
            CHECK(!fc::noalloc_two_pass(FC_SCHED_FUSED, true, K, bytes, 100, 0), "split K=%d", K);
            CHECK(!fc::noalloc_two_pass(FC_SCHED_RESIDENT, false, K, bytes, 257, 256), "resident K=%d", K);
            CHECK(fc::noalloc_two_pass(FC_SCHED_RESIDENT, false, K, bytes, 256, 256) == (bytes == 4 && K >= 8),
                  "resident, one tile a block, K=%d", K);
        }
}

// plans of several rounds that are resident
static void resident() {
    const uint64_t a = uint64_t(1) << 25, b = uint64_t(3) << 24, big = uint64_t(200) << 20;
    for (int K = 1; K <= 64; ++K)
        for (int bytes : {2, 4}) {
            const int row = K * bytes;
            CHECK(!fc::default_resident(K, bytes, 1, 1000, (64 << 20) - 1), "short step, K=%d", K);
            CHECK(fc::default_resident(K, bytes, 1, 1000, 64 << 20), "one round, K=%d", K);
            CHECK(fc::default_resident(K, bytes, 2, a - 1, big) == (row >= 48), "below 2^25, K=%d of %d", K, bytes);
            CHECK(fc::default_resident(K, bytes, 2, a, big) == (row >= 44), "2^25, K=%d of %d", K, bytes);
            CHECK(fc::default_resident(K, bytes, 2, b - 1, big) == (row >= 44), "below 3 * 2^24, K=%d of %d", K, bytes);
            CHECK(fc::default_resident(K, bytes, 2, b, big) == (row >= (bytes == 2 ? 32 : 40)), "3 * 2^24, K=%d of %d", K, bytes);
        }
}

// update-only launches with a thread per vector
static void sgd() {
    CHECK(fc::sgd_vector_per_thread(shape(64, 2)), "resident tiles of two vectors");
    for (int block : {64, 128, 256})
        for (int vecs : {1, 2, 4})
            CHECK(fc::sgd_vector_per_thread(shape(block, vecs)) == (block == 64 && vecs == 2), "(%d, %d)", vecs, block);
}

int main(int, char** argv) {
    const struct {
        const char* name;
        void (*run)();
    } rules[] = {{"copies", copies}, {"packed", packed}, {"shapes", shapes}, {"short_steps", short_steps}, {"split_plans", split_plans}, {"noalloc", noalloc},
                 {"resident", resident}, {"sgd", sgd}};
    for (const auto& r : rules)
        if (!std::strcmp(argv[1], r.name)) {
            r.run();
            if (!failures) std::printf("%s: as measured\n", r.name);
            return failures ? 1 : 0;
        }
    return 2;
}
