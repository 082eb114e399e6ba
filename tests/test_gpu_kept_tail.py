"""Clipped steps of which the memory-side cache keeps the end of the reduced gradient, so that sweep 2 begins with the last block."""
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, hp_dict, hp_struct, stream
import test_gpu_cache_policy as policy

pytestmark = pytest.mark.gpu
M = policy.M


# Of a gradient of more than 56 M elements the end is kept, and sweep 2 starts there; in a range of two chunks the line lies in the first.
@pytest.mark.parametrize("strategy,L,dtype", [("NNG", 56 * M, wl.BF16), ("NNG", 56 * M + 264, wl.F16), ("NNN", 29 * M + 8, wl.BF16),
                                              ("NNN", 29 * M + 8, wl.F32)])
def test_large_gradients(paro, strategy, L, dtype):
    policy.test_steps_at_the_limits(paro, 2, strategy, L, dtype)


@pytest.mark.parametrize("strategy,sizes", [
    ("NNN", [20 * M + 8, 1000, 39 * M + 3, 256]), ("NNG", [57 * M, 512, 56 * M + 256]), ("NNN", [3 * M + 1, 1000, 18 * M, 256])])
def test_exempt_tensors_and_both_layouts_give_the_same(paro, strategy, sizes):
    """Sweep 2 in one launch per chunk, from the first on; per-tensor gradients whose blocks start on cache lines, and not."""
    P, rank = 2, 1
    plan = paro.paro_plan(P, 1, strategy, sizes, no_decay=[i % 2 for i in range(len(sizes))])
    lay = orc.layout(P, 1, sizes)
    ob, ol = orc.state_range(lay, rank, strategy[2])
    contrib = [torch.zeros(P * lay.L, dtype=torch.bfloat16, device=DEV) for _ in range(P)]
    for q, x in enumerate(contrib):
        x[:sum(sizes)] = torch.randn(sum(sizes), generator=torch.Generator(device=DEV).manual_seed(q), device=DEV).mul_(0.01)
    off = [sum(sizes[:i]) for i in range(len(sizes))]
    whole = [[x[o:o + n].clone() for o, n in zip(off, sizes)] for x in contrib]
    tables = [torch.tensor([t.data_ptr() for t in w], dtype=torch.int64, device=DEV) for w in whole]
    start = [t.to(DEV) for t in wl.master_state(ol, 72)]
    results = []
    for ptrs, layout in (([x.data_ptr() + 2 * ob for x in contrib], paro.PARO_CHUNK), ([t.data_ptr() for t in tables], paro.PARO_TENSORS)):
        p, m, v = (t.clone() for t in start)
        g, ss = torch.empty(ol, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)
        dst = torch.zeros(orc.pack_slot(lay, rank, strategy)[0], dtype=torch.bfloat16, device=DEV)
        hp = hp_struct(paro, hp_dict(P, max_norm=0.1), 3)
        paro.paro_step_fused(plan, rank, ptrs, layout, hp, g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(),
                             dst.data_ptr(), stream())
        results.append((g, p, m, v, dst))
        exact = sum(float(g[i:i + 16 * M].double().square().sum()) for i in range(0, ol, 16 * M))
        assert abs(float(ss) - exact) <= 1e-11 * exact
    want = contrib[1].float() + contrib[0].float()
    assert torch.equal(results[0][0], want[ob:ob + ol])
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("P,G,L", [(2, 1, 32 * M), (2, 1, 32 * M + 8), (8, 4, 14 * M), (8, 4, 14 * M + 8)])
def test_all_gather_messages_of_which_the_start_is_kept(paro, P, G, L):
    plan = paro.paro_plan(P, G, "IIG", [P * L])
    bufs = [torch.randint(-30000, 30000, (P * L,), dtype=torch.int16, device=DEV) for _ in range(P)]
    want = torch.cat([bufs[paro.paro_owner_of_chunk(plan, c)][c * L:(c + 1) * L] for c in range(P)])
    steps = sorted({(m.phase, m.ring, m.step) for q in range(P) for m in paro.paro_schedule(plan, q, paro.PARO_AG)})
    for phase, ring, step in steps:
        for q in range(P):
            paro.paro_collective_step(plan, q, paro.PARO_SCHED_DEFAULT, paro.PARO_AG, phase, ring, step, [b.data_ptr() for b in bufs], stream())
    assert all(torch.equal(b, want) for b in bufs)
