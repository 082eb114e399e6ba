"""The weight-decay mask from the chunk's table (one entry per 256 elements, a bit per element where a block is mixed) and
from the tensors themselves: the same bits, over lists whose flags change inside words, at ends of blocks and in padding."""
import numpy as np
import pytest
import torch

from harness import DEV, hp_dict, hp_struct, np_of, stream

pytestmark = pytest.mark.gpu

LISTS = {
    "flags change inside a word": ([1, 2, 3, 4, 5, 250, 7, 31, 33, 1, 700, 13], [1, 0, 1, 0, 1, 0, 1, 0, 0, 1, 0, 1]),
    "at ends of blocks": ([256, 256, 255, 257, 512, 1, 255, 768], [0, 1, 1, 0, 1, 0, 1, 0]),
    "several exempt tensors fill a block": ([100, 156, 0, 256, 128, 64, 64, 300], [1, 1, 0, 0, 1, 1, 1, 0]),
    "everything exempt up to the padding": ([1000, 501], [1, 1]),
    "a block of 256 tensors": ([1] * 512 + [40], [i % 3 == 0 for i in range(513)]),
}


@pytest.mark.parametrize("clip", [True, False])
@pytest.mark.parametrize("strategy", ["IIG", "III"])
@pytest.mark.parametrize("name", LISTS)
def test_table_and_tensors_give_the_same_bits(paro, name, strategy, clip, monkeypatch):
    sizes, flags = LISTS[name]
    P, G, out = 2, 1, {}
    for route in ("table", "tensors"):
        if route == "tensors":
            monkeypatch.setenv("PARO_TILE_TABLE_MAX_TILES", "0")
        else:
            monkeypatch.delenv("PARO_TILE_TABLE_MAX_TILES", raising=False)
        plan = paro.paro_plan(P, G, strategy, sizes, no_decay=[int(f) for f in flags])
        for rank in range(P):
            ol = paro.paro_range(plan, rank, "O")[1]
            gen = torch.Generator(device=DEV).manual_seed(31 + rank)
            grads = [torch.randn(ol, generator=gen, device=DEV).to(torch.bfloat16) for _ in range(P)]
            p, m, v = (torch.randn(ol, generator=gen, device=DEV).abs_() for _ in range(3))
            old = p.clone()
            g = torch.zeros(ol, device=DEV)
            ss = torch.zeros(1, dtype=torch.float64, device=DEV)
            dst_len = paro.paro_pack_slot(plan, rank)[0]
            dst = torch.zeros(dst_len, dtype=torch.bfloat16, device=DEV)
            hp = dict(hp_dict(P, max_norm=1.0 if clip else 0.0), weight_decay=0.5)
            paro.paro_step_fused(plan, rank, [t.data_ptr() for t in grads], paro.PARO_CHUNK, hp_struct(paro, hp, 3), g.data_ptr(),
                                 ss.data_ptr(), p.data_ptr(), m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
            out[route, rank] = [np_of(x) for x in (p, m, v, dst)]
            assert not torch.equal(p, old)
    for rank in range(P):
        for a, b in zip(out["table", rank], out["tensors", rank]):
            np.testing.assert_array_equal(a, b)
