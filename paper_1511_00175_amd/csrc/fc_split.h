// Reduce and fused-step kernels for short steps: one tile is the work of a
// whole block, whose waves share the replicas.  Included by the translation
// units that instantiate them (fc_reduce_f32.hip, fc_reduce_f16.hip).
//
// With one wave per tile (reduce_kernel) a plan of few tiles leaves most of
// the chip idle, and each wave works through its K replicas batch after batch,
// one trip to memory each: time goes with K / batch, not with the bytes.
// Here a tile is 64 lanes of V = 1 or 2 elements and its block has up to 16
// waves, so that every replica byte of a step of a few tens of MB is asked
// for at once, from every compute unit.
//
// Tree order: wave q reduces replicas [q run, (q + 1) run) in registers, run a
// power of two, so that its sum is a complete subtree of the tree over all K
// (the last wave's may be shorter: the tree over its leaves is what the
// level-by-level pairing leaves of them).  The waves' sums meet in LDS, and
// the thread that owns an element pairs them level by level, an odd last one
// moving up unchanged: the same association as reduce_kernel, bit for bit.
//
// Linear order: the additions of one element are one serial chain, so only the
// loads are shared: the waves put batches of C replicas each into LDS, widened
// to fp32, and the element's owner adds them in order while the next batches
// are on their way.
//
// The element's owner (thread e of the block owns element e of the tile)
// loads w and v before the replicas and applies the update; a broadcast takes
// w' through LDS and spreads the K destinations over the waves.
#pragma once

#include "fc_device.h"

#pragma clang fp contract(off)

namespace fc {
namespace {

// V = 2 elements per lane: 8 bytes of fp32, 4 bytes of fp16
template <> struct Rep<FC_F32, 2> {
    typedef u2 raw;
    __device__ static __forceinline__ raw load(gptr_t base, uint32_t off) {
        return __builtin_bit_cast(u2, __builtin_amdgcn_raw_buffer_load_b64(rsrc((const void*)base), off, 0,
                                                                          CPOL_STREAM_LOAD));
    }
    __device__ static __forceinline__ void widen(const raw& r, float* x) {
        const f2 f = __builtin_bit_cast(f2, r);
        x[0] = f.x; x[1] = f.y;
    }
};
template <> struct Rep<FC_F16, 2> {
    typedef unsigned int raw;
    __device__ static __forceinline__ raw load(gptr_t base, uint32_t off) {
        return __builtin_amdgcn_raw_buffer_load_b32(rsrc((const void*)base), off, 0, CPOL_STREAM_LOAD);
    }
    __device__ static __forceinline__ void widen(const raw& r, float* x) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        const h2 h = __builtin_bit_cast(h2, r);
        x[0] = static_cast<float>(h.x); x[1] = static_cast<float>(h.y);
    }
};

constexpr int SPLIT_MAXD = 3;   // pending-subtree stack: runs of up to 4 batches

// The wave's vector of replicas [k, k + n), n <= SPLIT_C (nothing for n <= 0).
// All pointers are read first, at once (the table holds TABLE_PAD readable
// entries past the last replica), and the loads go out in groups of 4; the
// surplus of the last group re-reads the last replica.
template <int DT, int V>
__device__ __forceinline__ void load_batch(const void* const* grads, int k, int n, uint64_t start_bytes, uint32_t off,
                                           typename Rep<DT, V>::raw (&r)[SPLIT_C]) {
    if (n <= 0) return;
    gptr_t base[SPLIT_C];
#pragma unroll
    for (int j = 0; j < SPLIT_C; ++j) base[j] = gread(ldc(grads, k + j)) + start_bytes;
#pragma unroll
    for (int g = 0; g < SPLIT_C; g += 4) {
        if (g < n) {
#pragma unroll
            for (int j = g; j < g + 4; ++j) r[j] = Rep<DT, V>::load(base[j], off);
        }
    }
}

// The tree over the first n of N (a power of two) subtrees x[0], x[1], ...,
// level by level, an odd last one moving up unchanged; into x[0].
template <int N, int V> __device__ __forceinline__ void tree_of(float (&x)[N][V], int n) {
#pragma unroll
    for (int half = N / 2; half >= 1; half /= 2) {
#pragma unroll
        for (int m = 0; m < half; ++m)
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const float sum = x[2 * m][i] + x[2 * m + 1][i];
                x[m][i] = 2 * m + 1 < n ? sum : x[2 * m][i];
            }
        n = (n + 1) / 2;
    }
}

// The tree over the n <= N waves' sums of one element, p[0], p[T], p[2T], ...
template <int N, int T> __device__ __forceinline__ float tree_of_waves(const float* p, int n) {
    float x[N][1];
#pragma unroll
    for (int r = 0; r < N; ++r) x[r][0] = p[(r < n ? r : n - 1) * T];
    tree_of(x, n);
    return x[0][0];
}

// acc + p[0] + p[T] + p[2T] + ..., n >= 1 values one after another, read in
// batches of B: while one batch is added the next is read.  Reads go on to the
// end of the batch that holds the last value.
template <int T, int B> __device__ __forceinline__ void chain_read(const float* p, float (&x)[B]) {
#pragma unroll
    for (int j = 0; j < B; ++j) x[j] = p[j * T];
    // the scheduler would move these reads down to their first use
    __builtin_amdgcn_sched_barrier(0);
}
template <int B> __device__ __forceinline__ float chain_add(float acc, const float (&x)[B]) {
#pragma unroll
    for (int j = 0; j < B; ++j) acc = acc + x[j];
    return acc;
}
template <int B> __device__ __forceinline__ float chain_end(float acc, const float (&x)[B], int n) {
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const float sum = acc + x[j];
        acc = j < n ? sum : acc;
    }
    return acc;
}
template <int T, int B> __device__ __forceinline__ float chain(const float* p, int n, float acc) {
    float x[B], y[B];
    chain_read<T>(p, x);
    for (; n > 2 * B; n -= 2 * B) {
        chain_read<T>(p + B * T, y);
        acc = chain_add(acc, x);
        p += 2 * B * T;
        chain_read<T>(p, x);
        acc = chain_add(acc, y);
    }
    if (n > B) {
        chain_read<T>(p + B * T, y);
        acc = chain_add(acc, x);
        return chain_end(acc, y, n - B);
    }
    return chain_end(acc, x, n);
}

// One tile of ne <= 64 V elements; V: elements per lane of the replica loads.
// The block has at least V waves, so that thread e owns element e.
template <int DT, int V, bool TREE, int MODE>
__device__ __forceinline__ void split_tile(const ReduceArgs& a, int run, float* lds, uint64_t start, uint32_t ne,
                                           float lr_j, float wd_j) {
    constexpr uint32_t SG = DT == FC_F16 ? 2 : 4;
    constexpr int T = 64 * V;
    const int nw = static_cast<int>(blockDim.x) / 64;
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t e = threadIdx.x;
    const bool own = e < ne;
    const uint64_t start4 = start * 4;
    float w = 0.0f, v = 0.0f, s = 0.0f;
    if constexpr (MODE == MODE_STEP) {
        if (q < V) {
            const uint32_t off = (own ? e : 0u) * 4;
            ld32s<1>(gread(a.w) + start4, off, &w);
            ld32s<1>(gread(a.v) + start4, off, &v);
        }
    }
    const uint32_t roff = (lane * V < ne ? lane * V : 0u) * SG;  // ne is a multiple of V: lanes are whole
    typename Rep<DT, V>::raw r[SPLIT_C];
    if constexpr (TREE) {
        const int k0 = q * run;
        const int cnt = a.K - k0 < run ? a.K - k0 : run;
        const int full = cnt / SPLIT_C, rest = cnt % SPLIT_C;
        Acc<1, V> st[SPLIT_MAXD], sum;
        float x[SPLIT_C][V];
        for (int c = 0; c < full; ++c) {
#pragma unroll
            for (int j = 0; j < SPLIT_C; ++j)
                r[j] = Rep<DT, V>::load(gread(ldc(a.grads, k0 + c * SPLIT_C + j)) + start * SG, roff);
#pragma unroll
            for (int j = 0; j < SPLIT_C; ++j) Rep<DT, V>::widen(r[j], x[j]);
            tree_of(x, SPLIT_C);
#pragma unroll
            for (int i = 0; i < V; ++i) sum.a[0][i] = x[0][i];
            if (full > 1) push<SPLIT_MAXD>(st, sum, c);
        }
        if (rest || full > 1) {
            // a last batch that is not full is the newest subtree
            bool have = rest;
            if (full == 1) set(st[0], sum);
            if (rest) {
                load_batch<DT, V>(a.grads, k0 + full * SPLIT_C, rest, start * SG, roff, r);
#pragma unroll
                for (int j = 0; j < SPLIT_C; ++j) Rep<DT, V>::widen(r[j], x[j]);
                tree_of(x, rest);
#pragma unroll
                for (int i = 0; i < V; ++i) sum.a[0][i] = x[0][i];
            }
            fold<SPLIT_MAXD>(st, full, sum, have);
        }
#pragma unroll
        for (int i = 0; i < V; ++i) lds[q * T + lane * V + i] = sum.a[0][i];
        __syncthreads();
        if (q < V) {
            if (nw <= 4) s = tree_of_waves<4, T>(lds + e, nw);
            else if (nw <= 8) s = tree_of_waves<8, T>(lds + e, nw);
            else s = tree_of_waves<SPLIT_WAVES, T>(lds + e, nw);
        }
    } else {
        const int per = nw * SPLIT_C;  // replicas in LDS at a time
        s = -0.0f;                     // -0 + x is x, whatever x
        load_batch<DT, V>(a.grads, q * SPLIT_C, a.K - q * SPLIT_C, start * SG, roff, r);
        for (int c0 = 0; c0 < a.K; c0 += per) {
#pragma unroll
            for (int j = 0; j < SPLIT_C; ++j) {
                float x[V];
                Rep<DT, V>::widen(r[j], x);
#pragma unroll
                for (int i = 0; i < V; ++i) lds[(q * SPLIT_C + j) * T + lane * V + i] = x[i];
            }
            __syncthreads();
            const int k1 = c0 + per + q * SPLIT_C;
            load_batch<DT, V>(a.grads, k1, a.K - k1, start * SG, roff, r);
            if (q < V) s = chain<T, SPLIT_C>(lds + e, a.K - c0 < per ? a.K - c0 : per, s);
            __syncthreads();
        }
    }
    if constexpr (MODE == MODE_REDUCE) {
        if (own) st32r<1>(gwrite(a.out) + start4, e * 4, &s);
    } else {
        float wn, vn;
        sgd1(s, w, v, lr_j, a.mu, wd_j, a.c, wn, vn);
        if (own) {
            st32r<1>(gwrite(a.w) + start4, e * 4, &wn);
            st32r<1>(gwrite(a.v) + start4, e * 4, &vn);
            if (a.out) st32r<1>(gwrite(a.out) + start4, e * 4, &s);
        }
        if (a.dst) {
            // w' through the first T floats of LDS: column e was read by
            // thread e alone
            if (own) lds[e] = wn;
            __syncthreads();
            const int per = (a.K + nw - 1) / nw, k0 = q * per;  // the wave's destinations
            if (lane * V < ne) {
                float x[V];
#pragma unroll
                for (int i = 0; i < V; ++i) x[i] = lds[lane * V + i];
                settle<V>(x);
                st32_copies_shared<V>(a.dst, k0, k0 + per < a.K ? k0 + per : a.K, start4, lane * V * 4, x);
            }
        }
    }
}

template <int DT, int V, bool TREE, int MODE>
__global__ __launch_bounds__(64 * SPLIT_WAVES) void split_kernel(ReduceArgs a, int run) {
    extern __shared__ f4 slot_vecs[];
    float* lds = reinterpret_cast<float*>(slot_vecs);
    const Tile tile = ld_tile(a.tiles, blockIdx.x);
    float lr_j = 0.0f, wd_j = 0.0f;
    if constexpr (MODE == MODE_STEP) {
        const int j = static_cast<int>(tile.seg & SEG_MASK);
        lr_j = a.lr * ldc(a.mults, 2 * j);
        wd_j = a.wd * ldc(a.mults, 2 * j + 1);
    }
    if (!(tile.seg & TAIL_BIT)) split_tile<DT, V, TREE, MODE>(a, run, lds, tile.start, tile.count * 4, lr_j, wd_j);
    else split_tile<DT, 1, TREE, MODE>(a, run, lds, tile.start, tile.count, lr_j, wd_j);
}

// Linear order where a tile has a compute unit to itself: the time goes with the
// additions' serial chain, so wave 0 does nothing else.  The other waves put
// batches of SPLIT_C replicas into one of two LDS buffers, one barrier per
// buffer, while wave 0 adds the other one.  Tiles of 64 elements; element e is
// lane e of wave 0.  8274 x K=1000 fp32 takes 10.7 us per step, of which 2.5 an
// empty launch (12.2 while a block could take several tiles, and then 13.5 with
// waves that load and add in turn).  A dependent fp32
// addition alone takes 1.9-2.1 ns, with its operand from LDS in batches of 16
// 3.3-3.7; from K=640 to 1024 a replica more costs 5.7 ns with 1 or 64 tiles,
// the rest being the barriers and waits at each buffer, 7.7 with 128 tiles and
// 11.1 with 256, where the loads bound it.  Two batches per wave on their way
// instead of one, 32 values read from LDS at a time instead of 16, or one wait
// for each batch of reads changed nothing.
template <int DT, int MODE>
__global__ __launch_bounds__(64 * SPLIT_WAVES) void chain_kernel(ReduceArgs a) {
    extern __shared__ f4 slot_vecs[];
    float* lds = reinterpret_cast<float*>(slot_vecs);
    constexpr uint32_t SG = DT == FC_F16 ? 2 : 4;
    constexpr int T = 64;
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int nw = static_cast<int>(blockDim.x) / 64;
    const int per = (nw - 1) * SPLIT_C;  // replicas per buffer
    const int row = (q - 1) * SPLIT_C;   // of a loading wave
    const uint32_t lane = threadIdx.x & 63;
    const Tile tile = ld_tile(a.tiles, blockIdx.x);
    const uint32_t ne = tile.seg & TAIL_BIT ? tile.count : tile.count * 4;
    const uint64_t start4 = tile.start * 4;
    const bool own = lane < ne;
    const uint32_t e = own ? lane : 0u;
    float lr_j = 0.0f, wd_j = 0.0f, w = 0.0f, v = 0.0f;
    typename Rep<DT, 1>::raw r[SPLIT_C];
    if (q) {
        load_batch<DT, 1>(a.grads, row, a.K - row, tile.start * SG, e * SG, r);
    } else if constexpr (MODE == MODE_STEP) {
        const int j = static_cast<int>(tile.seg & SEG_MASK);
        lr_j = a.lr * ldc(a.mults, 2 * j);
        wd_j = a.wd * ldc(a.mults, 2 * j + 1);
        ld32s<1>(gread(a.w) + start4, e * 4, &w);
        ld32s<1>(gread(a.v) + start4, e * 4, &v);
    }
    float s = -0.0f;  // -0 + x is x, whatever x
    float* buf = lds;
    for (int c0 = 0; c0 < a.K; c0 += per) {
        if (q) {
#pragma unroll
            for (int j = 0; j < SPLIT_C; ++j) Rep<DT, 1>::widen(r[j], &buf[(row + j) * T + lane]);
            const int k1 = c0 + per + row;
            load_batch<DT, 1>(a.grads, k1, a.K - k1, tile.start * SG, e * SG, r);
        }
        // wave 0 added the buffer that is filled next before it came here
        __syncthreads();
        if (!q) s = chain<T, SPLIT_C>(buf + lane, a.K - c0 < per ? a.K - c0 : per, s);
        buf = buf == lds ? lds + per * T : lds;
    }
    if constexpr (MODE == MODE_REDUCE) {
        if (!q && own) st32r<1>(gwrite(a.out) + start4, e * 4, &s);
    } else {
        float wn, vn;
        sgd1(s, w, v, lr_j, a.mu, wd_j, a.c, wn, vn);
        if (!q && own) {
            st32r<1>(gwrite(a.w) + start4, e * 4, &wn);
            st32r<1>(gwrite(a.v) + start4, e * 4, &vn);
            if (a.out) st32r<1>(gwrite(a.out) + start4, e * 4, &s);
        }
        if (a.dst) {
            __syncthreads();  // buffers done with
            if (!q) lds[lane] = wn;
            __syncthreads();
            const int n = (a.K + nw - 1) / nw, k0 = q * n;  // the wave's destinations
            if (own) {
                float x = lds[lane];
                settle<1>(&x);
                st32_copies_shared<1>(a.dst, k0, k0 + n < a.K ? k0 + n : a.K, start4, e * 4, &x);
            }
        }
    }
}

// Allow the chain kernel `lds` bytes of dynamic LDS (a property of the kernel,
// set when a plan that runs it is created).
template <int DT> hipError_t prepare_chain_dt(size_t lds) {
    for (const void* kernel : {reinterpret_cast<const void*>(&chain_kernel<DT, MODE_REDUCE>),
                               reinterpret_cast<const void*>(&chain_kernel<DT, MODE_STEP>)}) {
        const hipError_t e =
            hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int DT>
hipError_t launch_split_dt(const Shape& sh, int mode, int grid, const ReduceArgs& a, hipStream_t s) {
    if (sh.chain) {
        return pick<MODE_REDUCE, MODE_STEP>(mode, [&](auto md) {
            hipLaunchKernelGGL((chain_kernel<DT, md.value>), dim3(grid), dim3(64 * sh.waves), split_lds(sh), s, a);
            return hipGetLastError();
        });
    }
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * sh.waves), split_lds(sh), s, a, sh.run);
        return hipGetLastError();
    };
    return pick<MODE_REDUCE, MODE_STEP>(mode, [&](auto md) {
        auto by_order = [&](auto v) {
            if (sh.tree) return go(&split_kernel<DT, v.value, true, md.value>);
            return go(&split_kernel<DT, v.value, false, md.value>);
        };
        return sh.lane == 2 ? by_order(I<2>{}) : by_order(I<1>{});
    });
}

}  // namespace
}  // namespace fc
