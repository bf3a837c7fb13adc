"""Default plans above 64 MiB: plans of several rounds are resident from 48 bytes
of replicas per parameter on, larger ones from 44, 40 or 32, and a one-round plan of few fp16
replicas runs its calls in one pass over the resident tiles, except a step
that broadcasts to more than 4 copies.  Reduce and step against the oracle, bit
for bit: the large plans on windows at the table's ends, its tails and the
borders of their rounds, the others on every element of a ragged table."""
import numpy as np
import pytest

from gpu_cases import LR, MU, WD, run_reduce, run_steps, same_bits
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc(device):
    import paper_1511_00175_amd as m
    return m


# schedules just below and from 2^25 parameters on, just below and from 3 * 2^24 on
@pytest.mark.parametrize("K,dtype,want", [(9, "f32", (1, 1, 1, 1)), (10, "f32", (1, 1, 1, 3)), (11, "f32", (1, 3, 3, 3)),
                                          (15, "f16", (1, 1, 1, 1)), (16, "f16", (1, 1, 1, 3)),
                                          (21, "f16", (1, 1, 1, 3)), (23, "f16", (1, 3, 3, 3))])
def test_several_rounds(fc, K, dtype, want):
    for n, sched in zip(((1 << 25) - 4, 1 << 25, (3 << 24) - 4, 3 << 24), want):
        p = fc.Plan([(0, n)], K, dtype, "tree")
        assert p.info().schedule == sched
        assert p.info().rounds >= 2 or sched == 1
        p.close()


@pytest.mark.parametrize("K,dtype,size", [(11, "f32", 1 << 25), (16, "f16", 3 << 24)])
def test_several_rounds_match_oracle(fc, K, dtype, size):
    import torch
    n = size + 4099
    rows = [(0, n - 70_000, 1.0, 1.0), ((n - 70_000 + 3) // 4 * 4, 70_001, 2.0, 0.0)]
    ext = rows[1][0] + rows[1][1]
    p = fc.Plan(rows, K, dtype, "tree")
    info = p.info()
    assert info.schedule == 3 and info.rounds >= 2
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    reps = torch.empty((K, (ext + 63) // 64 * 64), dtype=getattr(torch, {"f32": "float32", "f16": "float16"}[dtype]),
                       device="cuda").normal_(0, 0.01, generator=g)
    w = torch.empty(ext, device="cuda").normal_(0, 0.05, generator=g)
    v = torch.empty(ext, device="cuda").normal_(0, 1e-3, generator=g)
    w0, v0, out = w.clone(), v.clone(), torch.full((ext,), -1.0, device="cuda")
    p.tree_reduce(reps, out)
    p.step(reps, w, v, LR, MU, WD, 256)
    torch.cuda.synchronize()
    p.close()
    # windows of 2^17 elements at both ends and around every round's first tile
    tile = info.vecs_per_thread * 256
    starts = [0, rows[1][0] - 4096 * 8] + [-(-info.ntiles * r // info.rounds) * tile // 4 * 4 - (1 << 16)
                                           for r in range(1, info.rounds)]
    for a in starts:
        b = min(a + (1 << 17), ext)
        segs = [(max(o, a) - a, min(o + m, b) - max(o, a), x, y) for o, m, x, y in rows if o < b and o + m > a]
        win = [r[a:b].cpu().numpy() for r in reps]
        ew, ev, _, _ = oracle.step(segs, win, w0[a:b].cpu().numpy(), v0[a:b].cpu().numpy(), LR, MU, WD, 256)
        eo = oracle.tree_reduce(segs, win, out=np.full(b - a, -1.0, np.float32))
        assert same_bits(w[a:b].cpu().numpy(), ew) == 0 and same_bits(v[a:b].cpu().numpy(), ev) == 0, a
        assert same_bits(out[a:b].cpu().numpy(), eo) == 0, a
    del reps, w, v, w0, v0, out
    torch.cuda.empty_cache()


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
