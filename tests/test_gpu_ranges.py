"""Update ranges of several chunks (optimizer state sharded inside the group, or not at all), chunk
layout: one launch covers the whole range (large chunks of few ranks: one launch each), blocks are counted
from the range's start, and every chunk is folded in its own owner's order.  Sizes where that can go wrong: chunks shorter than a block (many
chunks in one block), a block more or less than a chunk, chunk ends inside a block, padding."""
import numpy as np
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, flat_inputs, hp_dict, hp_struct, np_of, oracle_update, run_rank, stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [8, 24, 248, 256, 264, 1000, 65544])
@pytest.mark.parametrize("P,G,strategy,sched,dtype", [
    (8, 2, "III", orc.HORING, wl.BF16), (6, 3, "NNN", orc.HRING, wl.F32), (8, 4, "NNI", orc.RING, wl.F16),
    (5, 5, "NNN", orc.RING, wl.BF16), (24, 2, "III", orc.HORING, wl.BF16), (4, 1, "III", orc.RING, wl.BF16)])
def test_every_chunk_of_the_range_in_its_own_order(paro, P, G, strategy, sched, dtype, L):
    _three_ranks(paro, P, G, strategy, sched, dtype, L, P * L - 3)           # the last chunk ends in padding


@pytest.mark.parametrize("L", [8, 24, 136])
@pytest.mark.parametrize("strategy,G,sched,dtype", [("III", 2, orc.HORING, wl.BF16), ("NNN", 6, orc.HRING, wl.F32)])
def test_chunks_that_are_all_padding(paro, strategy, G, sched, dtype, L):
    _three_ranks(paro, 24, G, strategy, sched, dtype, L, 24 * (L - 7))       # 7 elements a chunk short: whole chunks in the end


def _three_ranks(paro, P, G, strategy, sched, dtype, L, total):
    lay = orc.layout(P, G, [total])
    assert lay.L == L
    pl = paro.paro_plan(P, G, strategy, [total], sched=sched, grad_dtype=[dtype])
    n = P * lay.L
    dev, host = flat_inputs(P, n, 40 + L, dtype=dtype)
    for t, h in zip(dev, host):
        t[total:] = 0
        h[total:] = 0
    state = [np_of(t) for t in wl.master_state(n, 41 + L)]
    for a in state:
        a[total:] = 0
    for rank in sorted({0, P // 2, P - 1}):
        for max_norm in (0.0, 0.01):                                        # one sweep; two sweeps, clipped
            run_rank(paro, pl, lay, strategy, sched, rank, dev, host, state, hp_dict(P, max_norm=max_norm), 7,
                     check_unfused=max_norm > 0)


@pytest.mark.parametrize("P,G,strategy,sched,dtype", [
    (2, 1, "NNN", orc.RING, wl.BF16), (4, 2, "III", orc.HORING, wl.F16), (4, 4, "NNN", orc.RING, wl.BF16),
    (4, 2, "III", orc.HORING, wl.F32), (6, 3, "III", orc.HRING, wl.BF16)])
@pytest.mark.parametrize("L", [65528 * 256, 65529 * 256 + 8])
def test_large_chunks_with_few_ranks_are_launched_one_by_one(paro, P, G, strategy, sched, dtype, L):
    """Chunks of 65 536 blocks, counted with the one more that they may straddle and in eights, with up to 4 ranks and
    two-byte gradients; the others of that size are not.  The second size ends inside a block that two launches share."""
    total = P * L - 3
    lay = orc.layout(P, G, [total])
    assert lay.L == L
    pl = paro.paro_plan(P, G, strategy, [total], sched=sched, grad_dtype=[dtype])
    rank = P - 1
    ob, ol = orc.state_range(lay, rank, strategy[2])
    dev, host = flat_inputs(P, ol, 44, dtype=dtype)
    for t, h in zip(dev, host):
        t[total - ob:] = 0
        h[total - ob:] = 0
    state = [np_of(t) for t in wl.master_state(ol, 45)]
    g_ref, own_ref = orc.reduce_shard(lay, strategy, sched, rank, host, "chunk")
    ss_ref = orc.range_sumsq(lay, strategy, rank, g_ref)
    ptrs = [t.data_ptr() for t in dev]
    g = torch.empty(ol, dtype=torch.float32, device=DEV)
    ss, own = (torch.full((1,), -1.0, dtype=torch.float64, device=DEV) for _ in range(2))
    paro.paro_reduce_shard(pl, rank, ptrs, paro.PARO_CHUNK, g.data_ptr(), own.data_ptr(), stream())
    assert np_of(g).tobytes() == g_ref.tobytes()
    assert abs(float(own.item()) - own_ref) <= 1e-12 * own_ref
    hp = hp_dict(P, max_norm=0.01)
    lit = oracle_update(lay, strategy, rank, g_ref, *state, total_sumsq=ss_ref, hp=hp, step=3, literal32=True)
    dst_len, slot, n = orc.pack_slot(lay, rank, strategy)
    for static in (False, True):
        p, m, v = (torch.from_numpy(a.copy()).to(DEV) for a in state)
        g.zero_()
        dst = torch.zeros(dst_len, dtype=torch.bfloat16, device=DEV)
        tail = (hp_struct(paro, hp, 3), g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(),
                stream())
        if static:
            paro.paro_step_fused_static(pl, rank, ptrs, *tail)
        else:
            paro.paro_step_fused(pl, rank, ptrs, paro.PARO_CHUNK, *tail)
        assert np_of(g).tobytes() == g_ref.tobytes()
        assert abs(float(ss.item()) - ss_ref) <= 1e-12 * ss_ref
        for k, t in (("p", p), ("m", m), ("v", v)):
            assert np_of(t).tobytes() == lit[k].tobytes(), k
        assert np_of(dst)[slot:slot + n].tobytes() == lit["q"].tobytes()


@pytest.mark.parametrize("P,G,dtype,first", [
    (12, 6, wl.BF16, 131072), (32, 16, wl.F16, 65536), (64, 32, wl.BF16, 32768), (8, 4, wl.F32, 131072), (16, 8, wl.F32, 65536)])
@pytest.mark.parametrize("short", [16, 8, 7])
def test_more_ranks_where_chunks_begin_to_be_launched_one_by_one(paro, P, G, dtype, first, short):
    """`first`: the blocks of a chunk, counted with the one more that it may straddle and in eights, around which the sizes lie.  With 12 two-byte
    and 8 fp32 ranks each chunk is launched by itself from there on, 16 blocks short of it the range is one launch; with the others, for which
    there once were such lines, it is one launch on both sides (test_launch_rules says how many launches there are)."""
    L = (first - short) * 256 + (8 if short == 7 else 0)
    test_large_chunks_with_few_ranks_are_launched_one_by_one(paro, P, G, "III", orc.HORING, dtype, L)


@pytest.mark.parametrize("L", [(1 << 29) + 264, (1 << 29) + 30_000_008, (1 << 29) + 70_001_000])
def test_a_range_that_takes_several_launches_for_its_norm(paro, L):
    """The entry point that allocates nothing has room for the partial sums of 2^30 elements: a longer
    update range is swept in pieces whose sums are added in order.  Same results, the norm to the last bit, as with
    the plan's own scratch, which holds them all."""
    P = 2
    pl = paro.paro_plan(P, 1, "NNN", [P * L], grad_dtype=[wl.F32])
    n = P * L
    contrib = wl.chunk_contribs(P, n, 90, dtype=wl.F32, device=DEV)
    hp = hp_struct(paro, hp_dict(P, max_norm=0.01), 3)
    got = []
    for static in (True, False):
        p, m, v = wl.master_state(n, 91, device=DEV)
        g = torch.empty(n, dtype=torch.float32, device=DEV)
        ss = torch.zeros(1, dtype=torch.float64, device=DEV)
        dst = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
        ptrs = [t.data_ptr() for t in contrib]
        tail = (g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
        if static:
            paro.paro_step_fused_static(pl, 1, ptrs, hp, *tail)
        else:
            paro.paro_step_fused(pl, 1, ptrs, paro.PARO_CHUNK, hp, *tail)
        got.append((float(ss.item()), g, p, m, v, dst))
    assert got[0][0] == got[1][0] > 0
    assert all(torch.equal(a, b) for a, b in zip(got[0][1:], got[1][1:]))
