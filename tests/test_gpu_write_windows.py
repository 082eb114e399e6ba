"""Sweep 1 whose waves hold their results back for the chip's write windows, at both sides of the sizes where launches begin to:
the reduced gradient to the last bit, and its sum of squares, against the same adds in torch."""
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, hp_dict, hp_struct, stream

pytestmark = pytest.mark.gpu
TORCH = {wl.BF16: torch.bfloat16, wl.F16: torch.float16, wl.F32: torch.float32}


def _fold(paro, plan, contrib, chunk, lo, hi):
    order, group = paro.paro_fold_order(plan, chunk)
    total = None
    for k in range(0, len(order), group):
        part = contrib[order[k]][lo:hi].to(torch.float32, copy=True)
        for q in order[k + 1:k + group]:
            part += contrib[q][lo:hi]
        total = part if total is None else total + part
    return total


# Two-byte contributions of 12 ranks and more from 98 304 blocks on, 24 to 47 ranks from 49 152; fp32 ones from 16 384 on, with fewer
# than 48 ranks not from 65 536 to 131 071.  The last sizes end inside a block; in a range of two chunks of two-byte contributions, each a
# launch of its own, the second begins inside one.  A range that is one launch has windows from 16 384 blocks in all on, over two-byte
# contributions of up to 16 ranks from 65 536 on; below 16 384 it has all waves that fit, with more than 8 ranks.
@pytest.mark.parametrize("P,G,strategy,dtype,blocks,more", [
    (12, 4, "IGG", wl.BF16, 98304, 0), (12, 12, "IGG", wl.BF16, 98303, 8), (11, 11, "IGG", wl.BF16, 98304, 8),
    (16, 8, "IGG", wl.F16, 98303, 0), (24, 8, "IGG", wl.F16, 49151, 248), (24, 6, "IGG", wl.BF16, 49151, 0),
    (47, 47, "IGG", wl.BF16, 49152, 8), (100, 10, "IGG", wl.BF16, 98304, 8), (12, 4, "IGG", wl.F32, 16383, 8),
    (13, 13, "IGG", wl.F32, 16383, 0), (48, 8, "IGG", wl.F32, 65536, 8), (20, 4, "IGG", wl.F32, 65535, 0),
    (20, 4, "IGG", wl.F32, 65536, 0), (12, 6, "III", wl.F32, 131072, 8), (32, 16, "III", wl.BF16, 65536, 8),
    (12, 6, "III", wl.F32, 8191, 128), (12, 6, "III", wl.F32, 8191, 120), (16, 4, "III", wl.F32, 4096, 8), (20, 20, "NNN", wl.F32, 820, 24),
    (12, 6, "III", wl.BF16, 32768, 8), (16, 4, "III", wl.F16, 16383, 248), (17, 17, "NNN", wl.BF16, 964, 8), (17, 17, "NNN", wl.F16, 963, 24),
    (64, 8, "III", wl.BF16, 2050, 8), (32, 16, "III", wl.BF16, 131072, 8), (100, 50, "III", wl.BF16, 131072, 8),
    (9, 3, "III", wl.BF16, 5461, 80), (10, 5, "III", wl.F16, 8192, 0), (64, 32, "III", wl.BF16, 2000, 40)])
def test_reduced_gradient_and_its_norm(paro, P, G, strategy, dtype, blocks, more):
    L = blocks * 256 + more
    total = P * L - 5
    plan = paro.paro_plan(P, G, strategy, [total], grad_dtype=[dtype])
    lay, rank = orc.layout(P, G, [total]), P - 1
    ob, ol = orc.state_range(lay, rank, strategy[2])
    gen = torch.Generator(device=DEV).manual_seed(P * 1000 + blocks)
    contrib = []
    for q in range(P):
        x = torch.randn(ol, generator=gen, device=DEV).mul_(0.01).to(TORCH[dtype])
        x[max(total - ob, 0):] = 0
        contrib.append(x)
    g, ss = torch.full((ol,), -1.0, device=DEV), torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
    p, m, v = (torch.rand(ol, generator=gen, device=DEV) for _ in range(3))
    dst = torch.zeros(orc.pack_slot(lay, rank, strategy)[0], dtype=torch.bfloat16, device=DEV)
    hp = hp_struct(paro, hp_dict(P, max_norm=0.1), 3)
    want = torch.cat([_fold(paro, plan, contrib, (ob + lo) // L, lo, lo + L) for lo in range(0, ol, L)])
    norm = sum(float(want[lo:lo + (1 << 24)].double().square().sum()) for lo in range(0, ol, 1 << 24))
    for _ in range(2):
        g.fill_(-1.0)
        paro.paro_step_fused(plan, rank, [x.data_ptr() for x in contrib], paro.PARO_CHUNK, hp, g.data_ptr(), ss.data_ptr(), p.data_ptr(),
                             m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
        assert torch.equal(g.view(torch.int32), want.view(torch.int32))
        assert abs(float(ss) - norm) <= 1e-11 * norm


# The single sweep: 33 two-byte contributions or 16 fp32 ones and more, from 768 MB of them on, 40 and 20 from 512 MB, with more than 64 ranks 8 MB a
# rank, 32 two-byte ones from 1664 MB.  Over a range of several chunks 32 two-byte ones, and more than 48, from 16 384 blocks on, others of 28 and more from 768 MB; up to 96 without
# pauses.  Small ones have all waves that fit, up to 8192 blocks of a range of more than 12 two-byte ones, and 4096 or a few
# less otherwise.  It gives what the two calls give whose sweeps it joins.
@pytest.mark.parametrize("P,G,strategy,dtype,L", [
    (32, 8, "IGG", wl.BF16, 26 << 20), (32, 8, "IGG", wl.BF16, (26 << 20) - 8), (33, 11, "IGG", wl.F16, 12201616), (33, 11, "IGG", wl.BF16, 12201608),
    (32, 8, "IGG", wl.BF16, 3 << 22), (32, 8, "IGG", wl.BF16, (3 << 22) - 8), (31, 31, "IGG", wl.BF16, (3 << 22) + 264),
    (64, 16, "IGG", wl.F16, (1 << 22) + 8), (100, 10, "IGG", wl.BF16, 1 << 22), (100, 10, "IGG", wl.BF16, (1 << 22) - 8),
    (16, 4, "IGG", wl.F32, (3 << 22) + 200), (16, 4, "IGG", wl.F32, (3 << 22) - 8), (15, 5, "IGG", wl.F32, 3 << 22),
    (32, 8, "III", wl.BF16, (3 << 20) + 8), (32, 8, "III", wl.BF16, (3 << 20) - 8), (40, 40, "NNN", wl.BF16, 168 << 10),
    (24, 24, "NNN", wl.F32, (233 << 10) + 8), (32, 16, "III", wl.BF16, 2 << 20), (32, 16, "III", wl.F16, (2 << 20) - 264),
    (28, 14, "III", wl.BF16, 7190240), (28, 14, "III", wl.F16, 7190232), (27, 9, "III", wl.BF16, 5 << 20),
    (96, 48, "III", wl.BF16, (2 << 20) + 8), (98, 49, "III", wl.F16, (2 << 20) + 264),
    (16, 8, "III", wl.BF16, 1 << 20), (16, 8, "III", wl.F16, (1 << 20) + 8), (13, 13, "NNN", wl.BF16, 40 << 10), (64, 32, "IGG", wl.F32, 1 << 20),
    (12, 4, "IGG", wl.BF16, (1 << 20) + 8), (64, 32, "III", wl.F32, 1 << 19)])
@pytest.mark.parametrize("exempt", [False, True])
def test_single_sweep(paro, P, G, strategy, dtype, L, exempt):
    sizes = [P * L // 2 + 3, 1000, P * L - P * L // 2 - 1008]                # the last 5 elements are padding
    plan = paro.paro_plan(P, G, strategy, sizes, grad_dtype=[dtype] * 3, no_decay=[0, 1, 1] if exempt else None)
    lay, rank = orc.layout(P, G, sizes), P - 1
    assert lay.L == L
    ob, ol = orc.state_range(lay, rank, strategy[2])
    gen = torch.Generator(device=DEV).manual_seed(P * 7 + exempt)
    contrib = [torch.randn(ol, generator=gen, device=DEV).mul_(0.01).to(TORCH[dtype]) for _ in range(P)]
    start = [torch.rand(ol, generator=gen, device=DEV) for _ in range(3)]
    ptrs = [x.data_ptr() for x in contrib]
    hp = hp_struct(paro, hp_dict(P, max_norm=0.0), 3)
    results = []
    for joined in (False, True, True):
        p, m, v = (t.clone() for t in start)
        g = torch.empty(ol, device=DEV)
        dst = torch.zeros(orc.pack_slot(lay, rank, strategy)[0], dtype=torch.bfloat16, device=DEV)
        tail = (p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
        if joined:
            paro.paro_step_fused(plan, rank, ptrs, paro.PARO_CHUNK, hp, 0, 0, *tail)
        else:
            paro.paro_reduce_shard(plan, rank, ptrs, paro.PARO_CHUNK, g.data_ptr(), 0, stream())
            paro.paro_adam_shard(plan, rank, hp, g.data_ptr(), 0, *tail)
            want = torch.cat([_fold(paro, plan, contrib, (ob + lo) // L, lo, lo + L) for lo in range(0, ol, L)])
            assert torch.equal(g.view(torch.int32), want.view(torch.int32))
        results.append((p, m, v, dst))
    for other in results[1:]:
        assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(results[0], other))


# Per-tensor gradients: with 48 ranks and more sweep 1 runs all waves that fit from 16 384 blocks on (large chunks of fp32 ones see
# test_launch_rules).
@pytest.mark.parametrize("P,L,dtype", [(48, 1 << 22, wl.BF16), (48, (1 << 22) - 264, wl.BF16), (47, 1 << 22, wl.BF16), (64, (1 << 22) + 8, wl.F16), (48, 1 << 22, wl.F32)])
def test_tensors_of_many_ranks(paro, P, L, dtype):
    rank = P - 2
    ob, ol = orc.state_range(orc.layout(P, P, [P * L]), rank, "G")
    own = [L // 2 + 3, 1000, L - L // 2 - 1003]                             # the rank's chunk; every other is one tensor
    sizes = [L] * (ob // L) + own + [L] * (P - 1 - ob // L)
    plan = paro.paro_plan(P, P, "IGG", sizes, grad_dtype=[dtype] * len(sizes))
    gen = torch.Generator(device=DEV).manual_seed(P)
    contrib = [torch.randn(ol, generator=gen, device=DEV).mul_(0.01).to(TORCH[dtype]) for _ in range(P)]
    parts = [[t.clone() for t in torch.split(x, own)] for x in contrib]
    first = ob // L
    tables = [torch.tensor([w[t - first if first <= t < first + 3 else 0].data_ptr() for t in range(len(sizes))], dtype=torch.int64, device=DEV)
              for w in parts]                                               # tensors outside the range: an address that is never read
    g, ss = torch.full((ol,), -1.0, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)
    paro.paro_reduce_shard(plan, rank, [t.data_ptr() for t in tables], paro.PARO_TENSORS, g.data_ptr(), ss.data_ptr(), stream())
    want = _fold(paro, plan, contrib, first, 0, L)
    assert torch.equal(g.view(torch.int32), want.view(torch.int32))
    norm = float(want.double().square().sum())
    assert abs(float(ss) - norm) <= 1e-11 * norm
