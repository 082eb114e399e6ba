"""The weight-decay mask from the chunk's table (one entry per 256 elements, a bit per element where a block is mixed) and
from the tensors themselves: both bit for bit what the oracle's all-fp32 update gives, over lists whose flags change inside
words, at ends of blocks and in padding.  The table itself is compared element by element in test_decay_table_rule.py."""
import numpy as np
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, PtrTable, hp_dict, hp_struct, np_of, oracle_update, stream

pytestmark = pytest.mark.gpu

LISTS = {
    "flags change inside a word": ([1, 2, 3, 4, 5, 250, 7, 31, 33, 1, 700, 13], [1, 0, 1, 0, 1, 0, 1, 0, 0, 1, 0, 1]),
    "at ends of blocks": ([256, 256, 255, 257, 512, 1, 255, 768], [0, 1, 1, 0, 1, 0, 1, 0]),
    "several exempt tensors fill a block": ([100, 156, 0, 256, 128, 64, 64, 300], [1, 1, 0, 0, 1, 1, 1, 0]),
    "everything exempt up to the padding": ([1000, 501], [1, 1]),
    "a block of 256 tensors": ([1] * 512 + [40], [i % 3 == 0 for i in range(513)]),
}


@pytest.mark.parametrize("route", ["table", "tensors"])
@pytest.mark.parametrize("layout", ["chunk", "tensors"])
@pytest.mark.parametrize("strategy", ["IIG", "III"])
@pytest.mark.parametrize("name", LISTS)
def test_exempt_elements_are_the_oracles(paro, name, strategy, layout, route, monkeypatch):
    """Clipped steps and single sweeps.  (In the tensor layout the single sweep asks the tensors on either route.)"""
    if route == "tensors":
        monkeypatch.setenv("PARO_TILE_TABLE_MAX_TILES", "0")
    sizes, flags = LISTS[name]
    flags = [int(f) for f in flags]
    P, G = 2, 1
    lay = orc.layout(P, G, sizes)
    sched = orc.default_sched(P, G)
    plan = paro.paro_plan(P, G, strategy, sizes, no_decay=flags)
    bf16 = [wl.BF16] * len(sizes)
    sets = wl.tensor_contribs(P, sizes, bf16, 31, 1, device=DEV, align_elems=1)
    tables = [PtrTable(s.tensors) for s in sets]
    flat = [torch.cat([t.flatten() for t in s.tensors] + [torch.zeros(P * lay.L - lay.total, dtype=torch.bfloat16, device=DEV)])
            for s in sets]
    host = [[np_of(t) for t in s.tensors] for s in sets]
    state = [np.abs(np_of(t)) for t in wl.master_state(P * lay.L, 32)]
    for a in state:
        a[lay.total:] = 0
    for rank in range(P):
        ob, ol = orc.state_range(lay, rank, strategy[2])
        # the oracle's sum is over the rank's own chunk, the fused step's over all that the rank updates
        g_ref, _ = orc.reduce_shard(lay, strategy, sched, rank, host, "tensors")
        ss_ref = float((g_ref.astype(np.float64) ** 2).sum())
        old = [a[ob:ob + ol].copy() for a in state]
        if layout == "chunk":
            arrays = [x[ob:ob + ol].clone() for x in flat]
            ptrs, code = [x.data_ptr() for x in arrays], paro.PARO_CHUNK
        else:
            ptrs, code = [t.ptr() for t in tables], paro.PARO_TENSORS
        for max_norm in (0.01, 0.0):
            hp = dict(hp_dict(P, max_norm=max_norm), weight_decay=0.5)
            want = oracle_update(lay, strategy, rank, g_ref, *old, total_sumsq=ss_ref, hp=hp, step=3, no_decay=flags, literal32=True)
            all_decay = oracle_update(lay, strategy, rank, g_ref, *old, total_sumsq=ss_ref, hp=hp, step=3, literal32=True)
            assert want["p"].tobytes() != all_decay["p"].tobytes()
            p, m, v = (torch.from_numpy(a.copy()).to(DEV) for a in old)
            g = torch.zeros(ol, device=DEV)
            ss = torch.zeros(1, dtype=torch.float64, device=DEV)
            dst_len, slot, n = paro.paro_pack_slot(plan, rank)
            dst = torch.zeros(dst_len, dtype=torch.bfloat16, device=DEV)
            paro.paro_step_fused(plan, rank, ptrs, code, hp_struct(paro, hp, 3), g.data_ptr(), ss.data_ptr(), p.data_ptr(),
                                 m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
            what = f"rank {rank} clip {max_norm}"
            for k, t in (("p", p), ("m", m), ("v", v)):
                np.testing.assert_array_equal(np_of(t), want[k], err_msg=f"{what}: {k}")
            np.testing.assert_array_equal(np_of(dst)[slot:slot + n], want["q"], err_msg=what)


def test_the_limit_decides_the_route(paro, monkeypatch):
    """The table takes device memory: 36 bytes for each block of 256 here, all of them mixed, or none beyond the limit."""
    sizes = [128] * (1 << 19)
    flags = [k & 1 for k in range(len(sizes))]
    taken = {}
    for limit in ("", "0", "", "0"):                              # (twice: the first call of all also loads the code)
        if limit:
            monkeypatch.setenv("PARO_TILE_TABLE_MAX_TILES", limit)
        else:
            monkeypatch.delenv("PARO_TILE_TABLE_MAX_TILES", raising=False)
        plan = paro.paro_plan(1, 1, "NNN", sizes, no_decay=flags)
        L = paro.paro_shard_len(plan)
        p, m, v, g = (torch.zeros(L, device=DEV) for _ in range(4))
        paro.paro_pack_params(plan, 0, p.data_ptr(), torch.zeros(L, dtype=torch.bfloat16, device=DEV).data_ptr(), stream())
        torch.cuda.synchronize()                                  # the plan's other tables are made
        free = torch.cuda.mem_get_info()[0]
        paro.paro_adam_shard(plan, 0, hp_struct(paro, hp_dict(1), 3), g.data_ptr(), 0, p.data_ptr(), m.data_ptr(), v.data_ptr(), 0,
                             stream())
        torch.cuda.synchronize()
        taken[limit] = free - torch.cuda.mem_get_info()[0]
    assert taken[""] >= (L // 256) * 36 and taken["0"] < (L // 256) * 36
