"""The tensor layout's list of pieces: blocks with a tensor boundary inside are cut where the tensors meet
(from 5 ranks on, or in small chunks), up to 16 tensors a block; the others stay whole and are taken element
by element.  Boundaries at every position inside a group of four elements, tensors that end where a block
does, exactly 16 and more tensors in a block, padding after a cut; numbers of ranks on both sides of every
batch of loads; one and two blocks per wave.  Everything is compared bit for bit with the oracle's fold and
its all-fp32 update."""
import numpy as np
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, PtrTable, hp_dict, hp_struct, np_of, oracle_update, stream

pytestmark = pytest.mark.gpu

ONCE = [256, 255, 1, 1, 255, 257, 511] + [16] * 16 + [15] * 17 + [1] + [64] * 4 + [2, 254, 3, 253, 128, 129, 127] + \
    [0, 85, 86, 85, 0] + [1] * 40 + [216, 700, 4, 4, 4, 1300]


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 24, 33, 64])
def test_cut_blocks(paro, P, pairs, monkeypatch):
    if pairs:
        monkeypatch.setenv("PARO_PAIR_MIN_BLOCKS", "0")
    rng = np.random.default_rng(400 + P)
    sizes = []
    for k in range(P):                                            # every chunk gets the whole pattern, shifted
        sizes += [int(rng.integers(1, 256))] + ONCE + [3 + k]
    sizes += [5]                                                  # ... and the last one padding
    dtypes = [int(x) for x in rng.integers(0, 3, len(sizes))]
    no_decay = [int(x) for x in rng.integers(0, 2, len(sizes))]
    lay = orc.layout(P, 1, sizes)
    sched = orc.default_sched(P, 1)
    pl = paro.paro_plan(P, 1, "GGG", sizes, grad_dtype=dtypes, no_decay=no_decay)
    plain = paro.paro_plan(P, 1, "GGG", sizes, grad_dtype=dtypes)
    sets = wl.tensor_contribs(P, sizes, dtypes, 401 + P, 1, device=DEV, align_elems=1)
    tables = [PtrTable(s.tensors) for s in sets]
    host = [[np_of(t) for t in s.tensors] for s in sets]
    state = [np_of(t) for t in wl.master_state(P * lay.L, 402)]
    for a in state:
        a[lay.total:] = 0
    for rank in sorted({0, P // 2, P - 1}):
        ob, ol = orc.state_range(lay, rank, "G")
        g_ref, ss_ref = orc.reduce_shard(lay, "GGG", sched, rank, host, "tensors")
        old = [a[ob:ob + ol].copy() for a in state]
        for max_norm in (0.0, 0.01):
            for plan, mask in ((pl, no_decay), (plain, None)):
                hp = dict(hp_dict(P, max_norm=max_norm), weight_decay=0.1)
                lit = oracle_update(lay, "GGG", rank, g_ref, *old, total_sumsq=ss_ref, hp=hp, step=3, no_decay=mask,
                                    literal32=True)
                p, m, v = (torch.from_numpy(a.copy()).to(DEV) for a in old)
                g = torch.empty(ol, dtype=torch.float32, device=DEV)
                ss = torch.zeros(1, dtype=torch.float64, device=DEV)
                dst_len, slot, n = orc.pack_slot(lay, rank, "GGG")
                dst = torch.zeros(dst_len, dtype=torch.bfloat16, device=DEV)
                paro.paro_step_fused(plan, rank, [t.ptr() for t in tables], paro.PARO_TENSORS, hp_struct(paro, hp, 3),
                                     g.data_ptr(), ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(),
                                     stream())
                what = f"P {P} rank {rank} clip {max_norm} mask {mask is not None}"
                if max_norm:
                    assert np_of(g).tobytes() == g_ref.tobytes(), what
                    assert abs(float(ss.item()) - ss_ref) <= 1e-12 * ss_ref, what
                for k, t in (("p", p), ("m", m), ("v", v)):
                    assert np_of(t).tobytes() == lit[k].tobytes(), what + ": " + k
                assert np_of(dst)[slot:slot + n].tobytes() == lit["q"].tobytes(), what


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 8, 17])
def test_without_a_list(paro, P, pairs, monkeypatch):
    """The same where no list is built: every block found by a search, two of one tensor still taken together."""
    monkeypatch.setenv("PARO_TILE_TABLE_MAX_TILES", "0")
    test_cut_blocks(paro, P, pairs, monkeypatch)


@pytest.mark.parametrize("P,dtype,blocks", [(6, wl.BF16, 131072), (7, wl.BF16, 131072), (9, wl.BF16, 131072),
                                            (6, wl.F32, 131072), (9, wl.F32, 131072), (5, wl.F32, 262144)])
def test_boundaries_in_a_large_chunk(paro, P, dtype, blocks):
    """Many small tensors in a chunk of 131 072 blocks and more: with up to 6 ranks two blocks per wave and no cuts,
    with more blocks are cut, the list in address order; with fp32 gradients, which stream with up to 4 and more than 8
    ranks, cut with more than 4, but not from 262 144 blocks on."""
    sizes = wl.ragged_sizes(6200 * P * (blocks // 131072), seed=7)
    no_decay = [int(n % 3 == 0) for n in sizes]
    lay = orc.layout(P, 1, sizes)
    assert lay.L // 256 >= blocks
    sched, rank = orc.default_sched(P, 1), P // 2
    pl = paro.paro_plan(P, 1, "GGG", sizes, grad_dtype=[dtype] * len(sizes), no_decay=no_decay)
    ob, ol = orc.state_range(lay, rank, "G")
    off = np.concatenate([[0], np.cumsum(sizes)])                 # only the tensors that meet the rank's range exist
    meets = [t for t in range(len(sizes)) if off[t] < ob + ol and off[t + 1] > ob]
    first, span = int(off[meets[0]]), int(off[meets[-1] + 1] - off[meets[0]])
    flat = [wl.draw(span, 403 + q, dtype=dtype, device=DEV) for q in range(P)]

    def views(x):
        some = {t: x[int(off[t]) - first:int(off[t + 1]) - first] for t in meets}
        return [some.get(t) for t in range(len(sizes))]
    tables = [PtrTable(views(x)) for x in flat]
    host = [views(np_of(x)) for x in flat]
    g_ref, ss_ref = orc.reduce_shard(lay, "GGG", sched, rank, host, "tensors")
    state = wl.master_state(ol, 404, device=DEV)
    old = [np_of(t) for t in state]
    for max_norm in (0.0, 0.01):
        hp = dict(hp_dict(P, max_norm=max_norm), weight_decay=0.1)
        lit = oracle_update(lay, "GGG", rank, g_ref, *old, total_sumsq=ss_ref, hp=hp, step=3, no_decay=no_decay,
                            literal32=True)
        p, m, v = (t.clone() for t in state)
        g = torch.empty(ol, dtype=torch.float32, device=DEV)
        ss = torch.zeros(1, dtype=torch.float64, device=DEV)
        dst_len, slot, n = orc.pack_slot(lay, rank, "GGG")
        dst = torch.zeros(dst_len, dtype=torch.bfloat16, device=DEV)
        paro.paro_step_fused(pl, rank, [t.ptr() for t in tables], paro.PARO_TENSORS, hp_struct(paro, hp, 3), g.data_ptr(),
                             ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
        if max_norm:
            assert np_of(g).tobytes() == g_ref.tobytes()
            assert abs(float(ss.item()) - ss_ref) <= 1e-12 * ss_ref
        for k, t in (("p", p), ("m", m), ("v", v)):
            assert np_of(t).tobytes() == lit[k].tobytes(), f"clip {max_norm}: {k}"
        assert np_of(dst)[slot:slot + n].tobytes() == lit["q"].tobytes()
