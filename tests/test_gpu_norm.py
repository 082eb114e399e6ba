"""How the norm gets from sweep 1 to sweep 2 of the clipped fused step: every partial sum added up by
sweep 2's waves (up to 2048 blocks of 256 elements), eight slice sums (up to 131 072 blocks), or one
total.  Sizes at both ends of each range, clipped and with the skip on overflow; the total that the call
leaves behind is the same on a second run, and sweep 2's results are those of the split calls given it."""
import pytest
import torch

import workloads as wl
from harness import DEV, hp_dict, hp_struct, stream

pytestmark = pytest.mark.gpu

BLOCK = 256


@pytest.mark.parametrize("blocks", [1, 8, 9, 64, 65, 2040, 2048, 2049, 8193, 131072, 131073])
def test_total_and_update_at_the_edges_of_the_rule(paro, blocks):
    P, n = 2, chunk_of(blocks)
    pl = paro.paro_plan(P, 1, "NNG", [P * n])
    contrib = wl.chunk_contribs(P, n, 60 + blocks % 7, device=DEV)
    ptrs = [t.data_ptr() for t in contrib]
    hp = hp_struct(paro, dict(hp_dict(P, max_norm=0.01), skip_nonfinite=True), 3)
    totals, after = [], []
    for split in (False, False, True):
        p, m, v = wl.master_state(n, 61, device=DEV)
        g = torch.empty(n, dtype=torch.float32, device=DEV)
        ss = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
        dst = torch.zeros(P * n, dtype=torch.bfloat16, device=DEV)
        if split:
            ss.fill_(totals[0])
            paro.paro_reduce_shard(pl, 1, ptrs, paro.PARO_CHUNK, g.data_ptr(), 0, stream())
            paro.paro_adam_shard(pl, 1, hp, g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(),
                                 dst.data_ptr(), stream())
        else:
            paro.paro_step_fused(pl, 1, ptrs, paro.PARO_CHUNK, hp, g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(),
                                 v.data_ptr(), dst.data_ptr(), stream())
        totals.append(float(ss.item()))
        after.append([t.clone() for t in (g, p, m, v, dst)])
    exact = float(after[0][0].double().square().sum())
    assert abs(totals[0] - exact) <= 1e-12 * exact
    assert totals[0] == totals[1]
    for a in after[1:]:
        assert all(torch.equal(x, y) for x, y in zip(after[0], a))


@pytest.mark.parametrize("layout", ["chunk", "tensors"])
@pytest.mark.parametrize("blocks", [1, 8, 9, 65, 2047, 2048, 2049, 4099, 16384, 16385, 131072, 131073])
def test_the_reduce_call_leaves_the_fused_steps_total(paro, blocks, layout):
    """State sharded over all ranks: the fused step clips by the value that paro_reduce_shard gives, bit for bit."""
    P, n = 2, chunk_of(blocks)
    sizes = [n // 2 - 8, 8, P * n - n // 2]                   # three of them meet chunk 0
    pl = paro.paro_plan(P, 1, "NNG", sizes)
    contrib = wl.chunk_contribs(P, P * n, 64 + blocks % 7, device=DEV)
    if layout == "chunk":
        keep, kind = contrib, paro.PARO_CHUNK
    else:
        off = [0, sizes[0], sizes[0] + sizes[1], P * n]
        keep = [torch.tensor([t.data_ptr() + 2 * o for o in off[:3]], dtype=torch.int64, device=DEV) for t in contrib]
        kind = paro.PARO_TENSORS
    ptrs = [t.data_ptr() for t in keep]
    hp = hp_struct(paro, hp_dict(P, max_norm=0.01), 3)
    p, m, v = wl.master_state(n, 65, device=DEV)
    g = torch.empty(n, dtype=torch.float32, device=DEV)
    split, fused = (torch.full((1,), -1.0, dtype=torch.float64, device=DEV) for _ in range(2))
    dst = torch.zeros(P * n, dtype=torch.bfloat16, device=DEV)
    paro.paro_reduce_shard(pl, 0, ptrs, kind, g.data_ptr(), split.data_ptr(), stream())
    exact = float(g.double().square().sum())
    paro.paro_step_fused(pl, 0, ptrs, kind, hp, g.data_ptr(), fused.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(),
                         dst.data_ptr(), stream())
    assert abs(float(split.item()) - exact) <= 1e-12 * exact
    assert float(split.item()) == float(fused.item())


@pytest.mark.parametrize("blocks", [9, 2049, 131073])
def test_an_overflow_in_the_last_block_skips_the_step(paro, blocks):
    P, n = 2, chunk_of(blocks)
    pl = paro.paro_plan(P, 1, "NNG", [P * n])
    contrib = wl.chunk_contribs(P, n, 62, device=DEV)
    contrib[1][n - 1] = float("inf")
    hp = hp_struct(paro, dict(hp_dict(P, max_norm=0.01), skip_nonfinite=True), 3)
    p, m, v = wl.master_state(n, 63, device=DEV)
    before = [t.clone() for t in (p, m, v)]
    g = torch.empty(n, dtype=torch.float32, device=DEV)
    ss = torch.zeros(1, dtype=torch.float64, device=DEV)
    dst = torch.zeros(P * n, dtype=torch.bfloat16, device=DEV)
    paro.paro_step_fused(pl, 0, [t.data_ptr() for t in contrib], paro.PARO_CHUNK, hp, g.data_ptr(), ss.data_ptr(),
                         p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
    assert float(ss.item()) == float("inf")
    assert all(torch.equal(x, y) for x, y in zip(before, (p, m, v))) and not dst.any()


def chunk_of(blocks):
    """Elements of a chunk of that many blocks, the last one short."""
    return blocks * BLOCK - 8
