"""Default plans above 64 MiB: large plans of several rounds are resident from
32 bytes of replicas per parameter on, and a one-round plan of few fp16
replicas runs its calls in one pass over the resident tiles, except a step
that broadcasts to more than 4 copies; every call against the oracle, bit for
bit, on a ragged table."""
import numpy as np
import pytest

from gpu_cases import run_reduce, run_steps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


@pytest.mark.parametrize("K,dtype,below,above", [(7, "f32", 1, 1), (8, "f32", 1, 3), (11, "f32", 1, 3),
                                                 (15, "f16", 1, 1), (16, "f16", 1, 3), (23, "f16", 1, 3)])
def test_several_rounds(fc, K, dtype, below, above):
    for n, sched in (((1 << 25) - 4, below), (1 << 25, above)):
        p = fc.Plan([(0, n)], K, dtype, "tree")
        assert p.info().schedule == sched
        assert p.info().rounds >= 2 or sched == 1
        p.close()


@pytest.mark.parametrize("order", ["tree", "linear"])
@pytest.mark.parametrize("K", [1, 4, 5, 16])
def test_one_pass_fp16(fc, K, order):
    rows = [(0, 4_194_301, 1.0, 1.0), (4_194_304, 259, 2.0, 0.0), (4_194_564, 3, 1.0, 1.0)]
    p = fc.Plan(rows, K, "f16", order)
    info = p.info()
    assert (info.schedule, info.rounds) == (3, 1)
    # reduce and step launch a block per tile, not the persistent grid
    assert (info.grid, info.block_threads, info.k_waves) == (info.ntiles, 64, 1)
    p.close()
    rng = np.random.default_rng(K)
    bad, _, _ = run_reduce(fc, rows, K, "f16", order, rng, special=True)
    assert bad == 0
    assert run_steps(fc, rows, K, "f16", order, rng, steps=1, with_out=True, with_bcast=K in (4, 5)) == 0
