// Launch shapes and fc_step schedule chosen by default, and the (lane
// vectors, replicas per batch) pairs the kernels are compiled for.  These
// rules decide which kernel instance runs for a plan, so they live beside the
// device code.
#pragma once

#include <algorithm>
#include <cstdint>

#include "fc.h"
#include "fc_internal.h"

namespace fc {

// Launch-shape defaults, measured on MI355X for the five workloads:
//   fp16 replicas       : 4 vectors per lane, 4 replicas per batch, 256 threads
//   fp32, K <= 2        : 1 vector per lane, 8 replicas per batch, 256 threads
//         (K <= 4 below 2^23 parameters or with a capped grid)
//   fp32, 16 < K <= 64  : 4 vectors per lane, 2 replicas per batch, 256 threads
//   other fp32          : 1 vector per lane, 16 replicas per batch, 64 threads
// Four vectors per lane make every wave read 4 KiB of one replica at a time,
// which HBM serves better than 1 KiB pieces, as long as the lane's registers
// (16 accumulators per pending subtree) still allow enough waves in flight.
// With one or two replicas a wave has little to load: 4x fewer, larger blocks
// measured 1.3-5% faster on large plans (4 10^7 parameters, us per step, (1, 8,
// 256) vs (1, 16, 64): K=1 126.2 vs 127.6, K=2 155.9 vs 149.1 but its reduce
// 74.4 vs 84.8); from K=3 on one wave per block wins in every call of such
// plans (K=3 step 185.9 vs 176.4, broadcast 276 vs 261, reduce 105.7 vs 99.3;
// K=4 216 vs 203, 341 vs 318, 134 vs 125; equal at 1.4 10^7), but not of smaller
// ones (8000 x K=3 step 2.9 vs 3.3, 2^20 x K=3 reduce 3.4 vs 4.1, 4 10^6 x K=3
// 12.6 vs 13.4) nor where few blocks do all the work (65536 x K=4 reduce in 1
// block 54 vs 268).  Short steps of default
// plans have rules of their own (short_shape).
inline void default_shape(fc_dtype gdt, int K, uint64_t n_elems, bool capped, fc::Shape& sh) {
    if (gdt == FC_F16) {
        sh.vecs = 4; sh.kchunk = 4; sh.block = 256;
    } else if (K <= (capped || n_elems < (uint64_t(1) << 23) ? 4 : 2)) {
        sh.vecs = 1; sh.kchunk = 8; sh.block = 256;
    } else if (K > 16 && K <= 64) {
        sh.vecs = 4; sh.kchunk = 2; sh.block = 256;
    } else {
        sh.vecs = 1; sh.kchunk = 16; sh.block = 64;
    }
}

// (lane vectors, replicas per batch) of the resident kernel's tiles; with
// two vectors per lane K / kchunk must stay below 128 (stack depth 7).
inline bool resident_pair(int u, int c) { return (u == 1 && c == 16) || (u == 2 && c == 4); }

// Default resident tiles: fp32 replicas with K <= 16 take 2 lane-vectors and
// batches of 4 (each wave reads 2 KiB of a replica per tile), the others 1
// lane-vector and batches of 16.  Measured on MI355X with XCD-balanced
// shares, us per step, (1, 16) vs (2, 4): VGG-19 K=16 1871-1884 vs
// 1859-1862, 40 M x K=16 534.5 vs 512.0, 40 M x K=12 427.3 vs 417.0,
// 20 M x K=8 164.1 vs 161.4, 2^20 x K=16 14.8 vs 14.1, 2^23 x K=16 98.8 vs
// 99.3; for larger K the single vector with batches of 16 keeps more bytes
// in flight per register (GoogLeNet K=128 540 vs 548, AlexNet fp16 K=128
// 2611 vs 2705, NiN K=32 equal).
inline void default_resident_shape(fc_dtype gdt, int K, int& u, int& c) {
    if (gdt == FC_F32 && K <= 16) {
        u = 2; c = 4;
    } else {
        u = 1; c = 16;
    }
}
inline bool resident_fits_k(int u, int c, int K) { return u == 1 || K / c < 128; }

// Tiles per wave whose raw sums the resident kernel keeps in registers, on
// top of the LDS slots (the plan uses them only when they save rounds: the
// kernel instance that holds them is about 4x larger).  16 waves x 4 tiles
// per CU: fp32 replicas in tiles of 2 vectors (2 KiB of sums each) with
// batches of 4 and a depth-3 pending-subtree stack (K < 32; 123 VGPRs for
// the tree step, no spill), 1.8x the parameters of LDS alone per round;
// fp16 replicas in tiles of 1 vector (1 KiB) with batches of 16 and a stack
// of depth 5 (K < 512; 92 VGPRs), 1.4x.  Measured on MI355X (us per step):
// VGG-19 K=16 in 8 rounds instead of 14, 1792 vs 1829 on one machine, 1831-1836
// vs 1861-1887 on another; AlexNet fp16 K=128 in 5 rounds instead of 6,
// 2466.9 vs 2500.2 (both builds alternated in one process; 2469 vs 2496 in
// the parameter-server order).  Not kept: 5 or 6 fp16 tiles, which give
// AlexNet 4 rounds, 2497.8 and 2511.3 vs 2469.3 and 2468.9 with 4 tiles
// (the tree step's code: 43 KB with 4 tiles, 49 KB with 5, 57 KB with 6,
// against the 64 KB instruction cache two CUs share; which limit the larger
// instances hit was not measured); 12
// unrolled tiles (106 KB of code) and rolled ones (selects that cost load
// parallelism: AlexNet fp16 in 3 rounds 2571-2576 vs 2523-2529); fp32 tiles
// of 1 vector with K < 512, 4 per wave: VGG-19-sized K=32 in 10 rounds
// instead of 14, 3098.0 vs 3117.4, 60 M x K=32 1297.5 vs 1297.7.
inline int resident_rtiles(int gdt, int u, int c, int maxd) {
    if (gdt == FC_F16 && u == 1 && c == 16 && maxd <= 5) return 4;
    return gdt == FC_F32 && u == 2 && c == 4 && maxd <= 3 ? 4 : 0;
}

// Default shape of a step of less than RESIDENT_MIN_BYTES that one wave per
// tile serves (default_split says no).
//
// fp32: blocks of 256 threads and batches of 8 with few replicas (their one
// batch is nearly full, and a quarter of the blocks start the sooner) or, as the
// 4-vector shapes' successor, with more than 16; else one wave per block and
// batches of 16.  The larger blocks take 1024 elements each, so a plan of 1.2 or
// 3.1 of them per unit ends with most units idle: from 5 replicas on they serve
// plans whose last round of blocks is at least 80% full, or up to one block per
// unit.  Measured on MI355X, us, (1, 8, 256) / (1, 16, 64), data in the Infinity
// Cache: steps 2^18 x K=8 3.6 / 4.1, 520000 x K=8 5.2 / 5.3, 2^20 x K=8 8.2 / 8.5,
// but 300000 x K=8 with broadcast 6.1 / 5.1, 800000 x K=8 reduce 5.8 / 5.1; from 9
// replicas on two batches take longer: 300000 x K=16 5.8 / 5.1, 347457 x K=9 5.2 /
// 4.7, 2^18 x K=12 4.5 / 4.2.
//
// fp16: one wave per block and batches of 16 from 5 replicas on (2^20 x K=7 step
// 11.8 with (1, 8, 256), 7.3 with (1, 16, 64); its 4-vector shape 11.4 against 10.0
// at K=16).  Up to 4 replicas one wave's batch is nearly empty: the 4-vector
// shape serves plans of less than one of its blocks (1000 x K=1 reduce 2.3, 2.6
// with one-wave blocks) and those of more than 1536 tiles of 256 elements (800000
// x K=2 reduce 3.1 against 3.9), and between them blocks of 256 threads with
// batches of 8 for K <= 2 (100000 x K=1 1.3x the 4-vector shape's speed over all
// calls, one-wave blocks 1.2x), one-wave blocks for K = 3 and 4.  From 2^20
// elements on a step that also broadcasts would be up to 11% faster with the
// 4-vector shape (2^20 x K=12, data not in the cache, 18.2 / 20.3); its plain
// steps and reductions are 11 to 17% slower (11.1 / 9.9, 9.1 / 7.6), and a plan
// has one shape for all.
inline void short_shape(fc_dtype gdt, int K, int cus, uint64_t tiles256, uint64_t tiles1024, fc::Shape& sh) {
    const uint64_t cu = static_cast<uint64_t>(cus);
    const uint64_t places = (tiles1024 + cu - 1) / cu * cu;  // for blocks, over all rounds
    const bool filled = 10 * tiles1024 >= 8 * places;
    const bool larger = gdt == FC_F16 ? K <= 2
                        : K <= 4      ? true
                        : K <= 8      ? tiles1024 <= cu || filled
                                      : K > 16 && tiles1024 >= cu && filled;
    if (gdt == FC_F16 && K <= 4 && (tiles256 < 16 || tiles256 >= 1536)) {
        sh.vecs = 4; sh.kchunk = 4; sh.block = 256;
    } else if (larger) {
        sh.vecs = 1; sh.kchunk = 8; sh.block = 256;
    } else {
        sh.vecs = 1; sh.kchunk = 16; sh.block = 64;
    }
}

// The chain kernel (linear order, at most one tile per unit: wave 0 adds what the
// others load) from this many replicas on, and the LDS of its two buffers.  A
// replica costs 5.7 ns on up to 64 tiles, 3.3-3.7 of them the dependent addition
// with its operand from LDS, and 11 on 256 tiles, where the loads bound it; with
// fewer replicas the wave that does not load costs more than it saves.
// Measured on MI355X (us per call in a graph, split / chain): fp32 8274 x K=1000
// 13.5 / 12.2, 4096 x K=1000 12.1 / 10.3, 16384 x K=1000 14.4 / 13.9, 8000 x K=900
// with broadcast 16.2 / 14.1, fp16 4096 x K=700 10.2 / 9.3; 4096 x K=512 6.3 / 6.6,
// 16384 x K=128 3.4 / 3.7.
constexpr int CHAIN_MIN_K = 640;
constexpr int CHAIN_LDS = 2 * (SPLIT_WAVES - 1) * 16 * 64 * 4;

// The split kernel (a tile is a block's work, its waves share the replicas)
// for plans of few tiles of 256 elements per compute unit: one wave per tile, or
// a resident block's share of them, leaves most of the chip idle.
// With K <= 16 one wave asks for all replicas in one batch, and with K <= 32
// it does so in two, which two tiles per unit hide: those stay with one wave
// per tile.  Measured on MI355X (us per step in a HIP graph, before / now /
// the bytes at 7 TB/s): fp32 4096 x K=1000 59 / 6.5 / 2.4, 16384 x K=128 10.7
// / 2.8 / 1.2, 2^16 x K=64 39 / 5.0 / 2.5, 2^16 x K=256 20.3 / 12.0 / 9.7,
// 2^18 x K=128 24.9 / 23.8 / 19.8; fp16 16384 x K=1000 428 / 8.3 / 4.7, 2^16 x
// K=128 44 / 4.8 / 2.5, 2^18 x K=64 22 / 8.5 / 5.4; linear order fp32 8274 x
// K=1000 52 / 12.6 / 4.7, fp16 2^16 x K=128 58 / 5.7 / 2.5.
// How many tiles are few (split / resident, or one wave per tile below
// RESIDENT_MIN_BYTES; data not in the Infinity Cache): in tree order up to 4 per
// unit, where a step that broadcasts is the first to lose (fp16 300000 x K=200
// 76 / 69, 2^18 x K=200 64 / 66), and for fp32 from 400 replicas on up to 3 (2^18
// x K=512 93 / 82, 196608 x K=512 62 / 71); in linear order up to 5.5 (fp32
// 360000 x K=200 48.5 / 49.3, 393216 x K=1000 243 / 231), 4.5 for fp16, where the
// one wave that adds has the most to do (2^18 x K=400 36 / 45, 300000 x K=64 12.0,
// with one wave per tile 10.8).
//
// Tiles of 128 elements where that leaves two per unit (fp16: one, its rows
// are half as long), else of 64.  Tree: runs of 16 replicas, one batch, while
// that makes at most 32 waves' worth of 64-element tiles per unit, else of 32
// (2^18 x K=256 with runs of 32 / 64: 42.9 / 51.2; 2^16 x K=256 with 16 / 32:
// 13.0 / 12.0), and of 64 where that takes more than 8 waves (2^17 x K=400
// with 32 / 64: 36.5 / 34.0, K=512 43.5 / 42.2) or, in a narrower grid, 16.  Linear: as many waves as keep 4 KiB
// of each replica's row per unit in the block's batches, to the nearest power
// of two: more only wait for the one that adds (fp16 200000 x K=128 with 2 / 4
// waves 10.9 / 12.9, 2^16 x K=1000 with 4 / 8 24.6 / 22.2); the batches of all
// waves fit 64 KiB of LDS.
inline bool default_split(fc_dtype gdt, bool tree, int K, int cus, int lds_cu, uint64_t tiles256, uint64_t tiles128,
                          uint64_t tiles64, fc::Shape& sh) {
    const uint64_t cu = static_cast<uint64_t>(cus);
    const uint64_t half_units = tree ? (gdt == FC_F32 && K >= 400 ? 6 : 8) : gdt == FC_F16 ? 9 : 11;
    if (K <= 16 || 2 * tiles256 > half_units * cu || (K <= 32 && tiles256 >= 2 * cu)) return false;
    sh.lane = tiles128 >= (gdt == FC_F16 ? cu : 2 * cu) ? 2 : 1;
    const uint64_t width = sh.lane == 2 ? 2 * tiles128 : tiles64;  // the grid's width in 64-element tiles
    sh.run = 16;
    const int batches = (K + 15) / 16;
    if (tree) {
        const bool many = width * static_cast<uint64_t>(batches) > 32 * cu;
        if (many) sh.run = 32;
        while (sh.run < 64 && (K + sh.run - 1) / sh.run > (many ? SPLIT_WAVES / 2 : SPLIT_WAVES)) sh.run *= 2;
        sh.waves = (K + sh.run - 1) / sh.run;
    } else if (K >= CHAIN_MIN_K && tiles64 <= cu && lds_cu >= CHAIN_LDS) {
        sh.lane = 1;
        sh.chain = 1;
        sh.waves = 1 + std::min(batches, SPLIT_WAVES - 1);
    } else {
        const uint64_t budget = (gdt == FC_F16 ? 32 : 16) * cu;
        sh.waves = SPLIT_WAVES / sh.lane;
        // halve while the next smaller power of two is nearer (ratio above sqrt 2)
        while (sh.waves > sh.lane && 100 * width * static_cast<uint64_t>(sh.waves) > 141 * budget) sh.waves /= 2;
        sh.waves = std::min(sh.waves, std::max(batches, sh.lane));
    }
    sh.block = 64 * sh.waves;
    sh.vecs = 1;
    sh.kchunk = 16;
    return true;
}

// How many blocks share a tile's destinations in fc_broadcast on a plan that is
// not resident (1: the tile is one block's).  With few waves on the chip they
// are shared, at least 8 a block, until about 4096 waves store; with more the
// copies are bounded by the writes, and sharing makes them slower.  The split
// kernel's tiles have one wave each and K > 16 destinations; there the line is
// 2^18 elements.  Measured on MI355X, us, one block / shared, destinations in
// the Infinity Cache | not: 131072 x K=64 (128 waves) 15.1 / 6.1 | 14.9 / 6.8,
// 262144 x K=64 (256 waves) 15.8 / 9.7 | 15.6 / 13.4, 400000 x K=64 (391) 17.1 /
// 14.7 | 21.3 / 25.3, 600000 x K=64 19.9 / 20.4 | 28.9 / 37.8, 10^6 x K=16 9.3 /
// 9.3 | 14.6 / 16.7; one-wave blocks 100000 x K=200 (391) 11.7 / 11.7 | 12.3 /
// 14.5.
// A caller's cap on the grid (0: none) holds for every launch.
constexpr int BCAST_WAVES = 4096, BCAST_SHARE_WAVES = 256;
inline int bcast_groups(const Shape& sh, int K, int grid, uint64_t n_elems, int cap) {
    const int64_t waves = std::max<int64_t>(1, sh.lane ? grid : static_cast<int64_t>(grid) * (sh.block / 64));
    if (n_elems > (uint64_t(1) << 18) || (!sh.lane && waves > BCAST_SHARE_WAVES)) return 1;
    int64_t groups = std::min<int64_t>((K + 7) / 8, (BCAST_WAVES + waves - 1) / waves);
    if (cap > 0) groups = std::min<int64_t>(groups, cap / std::max(1, grid));
    return static_cast<int>(std::max<int64_t>(1, groups));
}

inline bool compiled_pair(int u, int c) {
    return (u == 1 && (c == 8 || c == 16)) || (u == 2 && (c == 8 || c == 16)) ||
           (u == 4 && (c == 2 || c == 4 || c == 8));
}

// The resident schedule (sums parked in LDS, one persistent grid, one launch
// per round) when one round of the grid holds the whole plan, or when a
// parameter's replicas take at least 48 bytes.  Measured on MI355X (us per
// step, resident vs the best other schedule): GoogLeNet K=128 543 vs 574,
// NiN K=32 162 vs 175, VGG-19 K=16 1926 vs 1979 and K=32 3323 vs 3567 (14
// rounds), AlexNet fp16 K=32/64/128 814/1379/2574 vs 890/1535/2579 and fp32
// K=32/64 1431/2553 vs 1473/2810 (6 rounds).  With w and v kept out of the
// Infinity Cache, at 48 bytes (fp32 K=12, fp16 K=24) resident wins at every
// size tried: 143.7 M fp32 1510 vs 1634, 61 M 661 vs 673, 20 M 214 vs 227,
// 2^25 366-384 vs 374-377; fp16 61 M 675 vs 711, 2^25 373 vs 383, 20 M 217
// vs 235.  At 40 bytes the two trade places by size (within 5%), and at 32
// bytes and below the fused kernel wins or ties (fp32 K=8: 61 M 492 vs 515,
// 2^25 275 vs 293-303, 20 M 165 vs 165; fp16 K=16: 2^25 282 vs 292; VGG-19
// K=4 766 vs 846), its update writes being a larger share of the bytes.
// Steps of less than RESIDENT_MIN_BYTES of algorithmic traffic (a few
// microseconds of HBM time) stay on the single-pass fused kernel, whose one
// round trip to memory beats the resident kernel's two phases: measured on
// MI355X, us per step in a HIP graph, fused vs resident: 2^20 x K=4 (33.5 MB)
// 5.2 vs 6.6, 60000 x K=128 (31 MB) 9.5 vs 10.1, 1000 x K=1024 36.8 vs 39.1;
// from 84 MB up the resident kernel is as fast or faster (2^20 x K=16 13.0
// vs 15.0, fp16 2^20 x K=64 24.1 vs 26.4, 2^21 x K=8 15.2 vs 15.6, 200000 x
// K=256 34.4 vs 34.2).
constexpr uint64_t RESIDENT_MIN_BYTES = uint64_t(64) << 20;
// Larger plans stay resident with fewer bytes of replicas: from 2^25 parameters
// on with 44, from 3 * 2^24 on with 32 in fp16 and 40 in fp32.  Measured on
// MI355X, us, fused vs resident, buffers not in the Infinity Cache: fp32 K=11
// 3.4 10^7 x step 333 vs 333, reduce 264 vs 251, broadcasting step 647 vs 593;
// fp16 K=23 349 vs 351, 277 vs 275, 1017 vs 900; fp32 K=10 6.1 10^7 x step 566 vs 563, reduce 434
// vs 420, 1.4 10^8 x step 1324 vs 1263; fp16 K=16 6.1 10^7 x step 489 vs 488,
// reduce 364 vs 345, 8 10^7 x step 642 vs 635, 1.4 10^8 x 1134 vs 1108.  Below
// the lines the step is what loses, its update writes being the larger share:
// fp32 K=8 3.4 10^7 x 262 vs 274, 4.5 10^7 x 349 vs 368, 6.1 10^7 x 478 vs 490,
// and at 1.4 10^8 x still 2.5% when the same buffers are used again; K=9 286 vs 296; K=10 4.5 10^7 x
// 414 vs 419; fp16 K=16 3.4 10^7 x 268 vs 277, K=20 313 vs 322.  Below 2^25 the
// 48 bytes hold: at 1.9 to 3.3 10^7 x fp32 K=8 to 11 and fp16 K=12 to 22 the
// resident step takes 0.96 to 1.06 times the fused one's time, and 1.03 to 1.16
// times on the same buffers again.  (So does a reduce below 6 10^7: fp16 K=23
// 3.4 10^7 x 256 vs 276, fp32 K=11 6.1 10^7 x 437 vs 459, the part of the
// replicas that stays in the cache being worth more to the fused kernel.)
constexpr uint64_t RESIDENT_44_ELEMS = uint64_t(1) << 25;
constexpr uint64_t RESIDENT_MANY_ELEMS = uint64_t(3) << 24;
inline bool default_resident(int K, int bytes_per_element, int64_t rounds, uint64_t n_elems, uint64_t step_bytes) {
    if (step_bytes < RESIDENT_MIN_BYTES) return false;
    const int64_t least = n_elems >= RESIDENT_MANY_ELEMS ? (bytes_per_element == 2 ? 32 : 40)
                          : n_elems >= RESIDENT_44_ELEMS ? 44
                                                         : 48;
    return rounds == 1 || static_cast<int64_t>(K) * bytes_per_element >= least;
}

// Calls that a default plan of one resident round runs in one pass, on the
// same tiles, with the reduce kernel: with few fp16 replicas a parameter's
// update moves as many bytes as its replicas, and a resident block's second
// phase waits for its slowest wave.  Measured on MI355X (us, resident vs one
// pass, steps): 2^22 x K=2 21.6 vs 16.2, x K=8 25.1 vs 22.4, x K=16 35.5 vs 32.6,
// 2^23 x K=4 42.2 vs 32.2, x K=16 67.5 vs 61.3, 1.4 10^7 x K=4 60.8 vs 55.3, x K=8
// 74.3 vs 73.2 (x K=12 92.2 vs 93.7, x K=16 106 vs 114; 2^23 x K=20 with the raw
// sum 85.4 vs 87.6); reduce 2^23 x K=2 21.2 vs 17.0, x K=8 28.8 vs 27.9.  A
// step's broadcast copies are written faster one destination at a time, but
// with up to 4 of them one pass still wins (2^23 x K=2 52.7 vs 44.2, x K=4 68.8
// vs 64.2, x K=8 96.9 vs 104).
inline bool one_pass_f16(int K, uint64_t n_elems) { return K <= (n_elems <= (uint64_t(1) << 23) ? 16 : 8); }
constexpr int ONE_PASS_BCAST_K = 4;

// fc_broadcast on a resident plan packs the tiles' descriptors into registers
// for its passes over the block's slots where a wave has more than two tiles
// (measured on MI355X, us, a load per tile / packed, destinations not in the
// Infinity Cache: fp16 plans 1.4 10^7 x K=4 58.2 / 52.0; a wave of one tile,
// packed slower: 4 10^5 x K=8 4.0 / 4.3).  Where the caller caps the grid, the
// blocks' own store rate is the bound and packing costs 5% (2^20 x K=128 in 64
// blocks 113.4 / 119.2).
inline bool bcast_packed(int K, int64_t ntiles, int64_t ranges, int cap) {
    return !cap && K >= 4 && ntiles > 2 * RESIDENT_WAVES * ranges;
}

// Resident launches record each block's rate (for fc_plan_balance) when a
// block's share of a round is at least this many tiles.  Measured on
// MI355X: the record costs about 0.6 us per launch (the timer read and the
// adds at the end of the reduce phase), 8% of a flat 2^20 x K=4 step (16
// tiles per block) and under 0.2% of the NiN-, GoogLeNet-, VGG-19- and
// AlexNet-sized steps (107-157 tiles per block), where balancing gains up to
// 1.6%.
constexpr int RESIDENT_RECORD_MIN_TILES = 32;

// Two passes (reduce into a raw-sum buffer, then update) when a parameter's
// replicas take more than 256 bytes: HBM serves the replica stream with one
// write stream far better than with two (measured on MI355X; see fc_schedule).
inline int default_schedule(int K, int bytes_per_element) {
    return static_cast<int64_t>(K) * bytes_per_element > 256 ? FC_SCHED_TWO_PASS : FC_SCHED_FUSED;
}

// fc_sgd_step on tiles of 64 lanes x 2 vectors (resident plans of few fp32
// replicas): one thread per vector, two waves per tile.  One wave took a tile's
// two vectors one after the other, and plans that became resident for their
// steps lost 5% here.  Measured on MI355X, us, one wave / two: 3.4 10^7
// parameters 115.9 / 110.7 (64-lane tiles of one vector 108.7), 1.4 10^8 467 / 440.
inline bool sgd_vector_per_thread(const Shape& sh) { return sh.vecs == 2 && sh.block == 64; }

// fc_step_noalloc in two passes with the raw sum in the library's fixed array:
// TWO_PASS plans of two launches, and where a schedule that the caller chose
// keeps the sum on chip more slowly than that: FUSED with more than 256 bytes
// of replicas per parameter, and RESIDENT fp32 plans of 8 replicas and more with
// at most one tile per block.  Measured on MI355X, us, on chip / two passes: FUSED
// fp16 4 10^6 x K=1000 1660 / 1229, fp32 1.4 10^7 x K=128 1223 / 1139; RESIDENT
// 65536 x K=16 7.5 / 6.4, 4000 x K=1000 65 / 58 (fp16 65.6 / 65.1, and 400000 x K=8
// 8.1 / 9.9).
inline bool noalloc_two_pass(int schedule, bool split, int K, int bytes_per_element, int ntiles, int blocks) {
    if (split) return false;
    if (schedule == FC_SCHED_RESIDENT) return bytes_per_element == 4 && K >= 8 && ntiles <= blocks;
    return schedule == FC_SCHED_TWO_PASS || default_schedule(K, bytes_per_element) == FC_SCHED_TWO_PASS;
}

}  // namespace fc
