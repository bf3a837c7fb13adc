"""Broadcast copies: worker counts around the batches of 8 pointers and the 16
from which they are used, destinations shared among blocks (few tiles), among
the waves of a split plan, and with the grid capped, by fc_broadcast and by the
step, against the oracle; nothing else is written."""
import numpy as np
import pytest

from gpu_cases import alloc_len, run_steps, same_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


ROWS = [(0, 3, 1.0, 1.0), (4, 700, 2.0, 0.0), (704, 65, 1.0, 1.0), (772, 2049, 1.0, 1.0)]


@pytest.mark.parametrize("max_blocks", [0, 3])
@pytest.mark.parametrize("K", [1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 130, 1000])
def test_copies(fc, K, max_blocks):
    import torch
    n = alloc_len(ROWS)
    src = np.random.default_rng(K).standard_normal(n).astype(np.float32)
    for opts in (dict(max_blocks=max_blocks), dict(max_blocks=max_blocks, schedule=1), dict(max_blocks=max_blocks, schedule=2)):
        plan = fc.Plan(ROWS, K, "f32", "tree", **opts)
        dst = torch.full((K + 1, n), -2.0, device="cuda")  # the last row belongs to nobody
        plan.broadcast(to_dev(src), dst[:K])
        got = dst.cpu().numpy()
        plan.close()
        expect = np.full(n, -2.0, np.float32)
        for off, m, _, _ in ROWS:
            expect[off:off + m] = src[off:off + m]
        assert sum(same_bits(got[k], expect) for k in range(K)) == 0, opts
        assert (got[K] == -2.0).all(), opts
    assert run_steps(fc, ROWS, K, "f16", "tree", np.random.default_rng(K), steps=1, with_bcast=True,
                     opts=dict(max_blocks=max_blocks)) == 0
