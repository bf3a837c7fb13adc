"""The split kernel (a tile is a block's work, its waves share the replicas),
which short plans of more than 16 workers run, against the oracle bit for bit:
worker counts at the edges of its batches (16), runs (16, 32, 64) and waves
(16), tile widths of 64 and 128 elements with lengths around them, tails, both
orders and storage types, a cap on the grid that its tiles do not reach, special
values, every optional output, and the raw sum written over a replica; for the
chain kernel too, where one wave adds what the others load."""
import numpy as np
import pytest

from gpu_cases import LR, MU, WD, alloc_len, host_replicas, run_reduce, run_steps, same_bits, to_dev
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


def rows_of(lengths):
    rows, off = [], 0
    for i, n in enumerate(lengths):
        rows.append((off, n, 2.0, 0.0) if i % 3 == 1 else (off, n, 1.0, 1.0))
        off = (off + n + 3) // 4 * 4 + 4 * (i % 2)
    return rows


# few tiles: 64 elements wide
NARROW = rows_of([1, 3, 4, 63, 64, 65, 127, 128, 130, 255, 257, 1000, 7])
# more than 512 tiles of at most 128 elements, most of them short
WIDE = rows_of([(5, 128, 17, 131, 64)[i % 5] for i in range(430)])


def tiles(rows, width):
    return sum(-(-(n // 4) // (width // 4)) + (1 if n % 4 else 0) for _, n, _, _ in rows)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("order", ["tree", "linear"])
@pytest.mark.parametrize("K", [17, 31, 33, 48, 128, 129, 256, 257, 512, 513, 639, 640, 1000, 1024])
def test_narrow_tiles_match_oracle(fc, K, order, dtype):
    p = fc.Plan(NARROW, K, dtype, order)
    info = p.info()
    p.close()
    assert (info.ntiles, info.kchunk, info.scratch_bytes) == (tiles(NARROW, 64), 16, 0)
    assert 2 <= info.block_threads // 64 <= 16
    # what the plan reports is the launch: the waves that share a tile, and their LDS
    assert info.k_waves == info.block_threads // 64
    chain = order == "linear" and K >= 640
    rows = 2 * 16 * (info.k_waves - 1) if chain else info.k_waves * (1 if order == "tree" else 16)
    assert info.lds_bytes == rows * 64 * 4
    rng = np.random.default_rng(K)
    bad, _, _ = run_reduce(fc, NARROW, K, dtype, order, rng, special=True)
    assert bad == 0
    assert run_steps(fc, NARROW, K, dtype, order, rng, steps=2, with_out=K % 2 == 0, with_bcast=K < 300) == 0


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("order", ["tree", "linear"])
@pytest.mark.parametrize("K,max_blocks", [(33, 0), (100, 0), (200, 0), (33, 5000)])
def test_wide_tiles_match_oracle(fc, K, max_blocks, order, dtype):
    p = fc.Plan(WIDE, K, dtype, order, max_blocks=max_blocks)
    info = p.info()
    p.close()
    assert (info.ntiles, info.kchunk) == (tiles(WIDE, 128), 16)
    assert info.grid == info.ntiles
    rng = np.random.default_rng(K)
    opts = dict(max_blocks=max_blocks)
    bad, _, _ = run_reduce(fc, WIDE, K, dtype, order, rng, opts=opts, special=True)
    assert bad == 0
    assert run_steps(fc, WIDE, K, dtype, order, rng, steps=2, opts=opts, with_out=True, with_bcast=K < 150) == 0


# few enough tiles for the chain kernel (linear order, at most one tile of 64
# elements per compute unit), with tails of one to three elements
CHAIN = rows_of([2000, 1, 65, 64, 3, 130, 4, 62, 259])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("K", [640, 655, 1000, 1024])
def test_chain_with_every_output(fc, K, dtype):
    """One wave adds, the others load into two buffers in turn; w' goes through
    one of them to the waves that share the copies."""
    p = fc.Plan(CHAIN, K, dtype, "linear")
    info = p.info()
    p.close()
    assert (info.ntiles, info.k_waves, info.lds_bytes) == (tiles(CHAIN, 64), 16, 2 * 15 * 16 * 64 * 4)
    rng = np.random.default_rng(K)
    assert run_steps(fc, CHAIN, K, dtype, "linear", rng, steps=2, with_out=True, with_bcast=True) == 0
    assert run_steps(fc, CHAIN, K, dtype, "linear", rng, steps=1, special=True) == 0


@pytest.mark.parametrize("order,K", [("tree", 70), ("linear", 70), ("linear", 700)])
def test_step_with_its_sum_over_a_replica(fc, order, K):
    import torch
    n = alloc_len(CHAIN)
    rng = np.random.default_rng(K)
    reps = host_replicas(rng, K, n, np.float32, scale=0.01)
    w = rng.standard_normal(n, dtype=np.float32)
    v = rng.standard_normal(n, dtype=np.float32) * np.float32(1e-3)
    for k in (0, 15, 16, K - 1):
        out = reps[k].copy()
        ew, ev, _, _ = oracle.step(CHAIN, list(reps), w, v, LR, MU, WD, 256, order=order, out=out)
        d, wd, vd = to_dev(reps), to_dev(w), to_dev(v)
        plan = fc.Plan(CHAIN, K, "f32", order)
        plan.step(d, wd, vd, LR, MU, WD, 256, out=d[k])
        torch.cuda.synchronize()
        plan.close()
        assert same_bits(wd.cpu().numpy(), ew) == 0 and same_bits(vd.cpu().numpy(), ev) == 0, k
        assert same_bits(d[k].cpu().numpy(), out) == 0, k


@pytest.mark.parametrize("order", ["tree", "linear"])
def test_sum_over_a_replica(fc, order):
    K = 70
    n = alloc_len(NARROW)
    reps = host_replicas(np.random.default_rng(3), K, n, np.float32)
    for k in (0, 16, K - 1):
        expect = oracle.tree_reduce(NARROW, list(reps), order=order, out=reps[k].copy())
        d = to_dev(reps)
        plan = fc.Plan(NARROW, K, "f32", order)
        plan.tree_reduce(d, d[k])
        assert same_bits(d[k].cpu().numpy(), expect) == 0
        plan.close()
