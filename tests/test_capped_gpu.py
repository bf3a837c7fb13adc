"""max_blocks: the shapes and kernels for short plans, which spread a plan over
many small blocks, serve a default plan only where the cap does not reach their
tiles; a grid capped below them keeps the larger tiles (and the persistent
blocks of a resident plan), which a block works through several times as fast.
Results against the oracle, bit for bit."""
import numpy as np
import pytest

from gpu_cases import LR, MU, WD, run_reduce, run_steps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


@pytest.mark.parametrize("n,K,dtype,order,cap,shape", [
    (4096, 17, "f32", "linear", 1, (256, 4, 2)), (65536, 17, "f16", "linear", 1, (256, 4, 4)),
    (65536, 64, "f32", "tree", 8, (256, 4, 2)), (300_000, 2, "f16", "tree", 8, (256, 4, 4)),
    (300_000, 17, "f16", "tree", 256, (256, 4, 4)), (200_000, 8, "f32", "tree", 32, (64, 1, 16)),
    # caps at the tiles of short plans and below: 64 of 64, 16 and 1172 of 256 elements
    (4096, 17, "f32", "tree", 64, (128, 1, 16)), (4096, 17, "f32", "tree", 63, (64, 1, 16)),
    (300_000, 7, "f16", "tree", 1172, (64, 1, 16)), (300_000, 7, "f16", "tree", 1171, (256, 4, 4))])
def test_shapes_under_a_cap(fc, n, K, dtype, order, cap, shape):
    p = fc.Plan([(0, n)], K, dtype, order, max_blocks=cap)
    info = p.info()
    p.close()
    assert (info.block_threads, info.vecs_per_thread, info.kchunk) == shape
    assert info.grid <= cap
    rows = [(0, n // 8 + 3, 1.0, 1.0), (n // 8 // 4 * 4 + 8, 70, 2.0, 0.0)]
    rng = np.random.default_rng(K)
    assert run_reduce(fc, rows, K, dtype, order, rng, opts=dict(max_blocks=cap))[0] == 0
    assert run_steps(fc, rows, K, dtype, order, rng, steps=1, opts=dict(max_blocks=cap), with_out=True,
                     with_bcast=True) == 0


@pytest.mark.parametrize("cap,resident", [(128, True), (16383, True), (16384, False)])
def test_one_pass_under_a_cap(fc, cap, resident):
    """A default plan of one resident round and few fp16 replicas runs one wave
    per tile only where the cap allows a block per tile: its persistent launches
    leave a record for fc_plan_balance, the others none."""
    import torch
    n, K = 1 << 22, 4
    p = fc.Plan([(0, n)], K, "f16", "tree", max_blocks=cap)
    assert p.info().schedule == 3 and p.info().rounds == 1
    reps = torch.zeros((K, n), dtype=torch.float16, device="cuda")
    w, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    p.step(reps, w, v, LR, MU, WD, 256)
    assert (max(p.balance()) > 0) == resident
    p.close()
