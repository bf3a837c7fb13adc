"""fc_step_noalloc runs the plan's own schedule (the two-pass plan keeps its raw
sum in the library's fixed array, the others on chip), or two passes where those
are faster (fused with many replicas, resident with one tile per block): each
against fc_step and the oracle, bit for bit, two calls in a row, the second smaller,
with and without a buffer for the raw sum."""
import numpy as np
import pytest

from test_zz_no_alloc import big_table, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


@pytest.mark.parametrize("with_out", [False, True])
@pytest.mark.parametrize("K,dtype,order,opts", [
    (20, "f32", "tree", dict(schedule=1)), (20, "f32", "linear", dict(schedule=2)), (70, "f16", "tree", dict(schedule=2)),
    (20, "f32", "tree", dict(schedule=3)), (9, "f16", "linear", dict(schedule=4, max_blocks=2)),
    (70, "f32", "tree", None), (40, "f16", "linear", None), (70, "f32", "tree", dict(schedule=1)),
    (16, "f32", "tree", dict(schedule=3)), (130, "f32", "linear", dict(schedule=3))])
def test_every_schedule(fc, K, dtype, order, opts, with_out):
    rng = np.random.default_rng(K)
    for n in (90_000, 20_000):
        segs = big_table(rng, n, dtype)
        vs_step, vs_oracle = run_both(fc, segs, K, dtype, order, rng, opts=opts, with_out=with_out)
        assert vs_step == 0 and vs_oracle == 0, (n, vs_step, vs_oracle)
