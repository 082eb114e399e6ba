"""Single sweeps (no clipping) at both sides of the sizes where the launch takes another form."""
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, hp_dict, hp_struct, np_of, run_rank, stream
from test_gpu_cache_policy import _Shifted

pytestmark = pytest.mark.gpu


# Over one chunk, waves pause where the launch reads 21 (one rank: 20) to 30.5 MB with 1 to 3 ranks: 14, 16, 18, 20 and 24 bytes an
# element here.
@pytest.mark.parametrize("P,dtype,L", [
    (2, wl.BF16, 1312496), (2, wl.BF16, 1312504), (2, wl.F16, 1906248), (2, wl.BF16, 1906256), (3, wl.BF16, 1166664),
    (3, wl.BF16, 1166672), (2, wl.F32, 1049992), (2, wl.F32, 1050000), (3, wl.F32, 1270832), (3, wl.F32, 1270840),
    (1, wl.BF16, 1428568), (1, wl.F16, 1428576), (1, wl.BF16, 2178568), (1, wl.BF16, 2178576), (1, wl.F32, 1600008), (4, wl.BF16, 1200008)])
def test_one_chunk(paro, P, dtype, L):
    lay = orc.layout(P, 1, [P * L])
    plan = paro.paro_plan(P, 1, "IIG", [P * L], sched=orc.RING, grad_dtype=[dtype])
    _last_rank(paro, plan, lay, P, dtype, orc.RING, "IIG")


def _last_rank(paro, plan, lay, P, dtype, sched, strategy):
    rank = P - 1
    ob, ol = orc.state_range(lay, rank, strategy[2])
    dev = wl.chunk_contribs(P, ol, 80 + P, dtype=dtype, device=DEV)
    padded = [_Shifted(t, ob) for t in dev]
    host = [_Shifted(np_of(t), ob) for t in dev]
    state = [_Shifted(np_of(t), ob) for t in wl.master_state(ol, 81)]
    run_rank(paro, plan, lay, strategy, sched, rank, padded, host, state, hp_dict(P, max_norm=0.0), 5, check_unfused=False)


# A range of g chunks: waves pause where the launch reads 19.5 to 31 MB (two ranks: 27), with up to 8 two-byte or 4 fp32 contributions.
# With two-byte ones it has fewer waves from 81 920 blocks times ranks on.
@pytest.mark.parametrize("P,G,sched,dtype,ol", [
    (2, 1, orc.RING, wl.BF16, 10485504), (2, 1, orc.RING, wl.BF16, 10485760), (4, 2, orc.HORING, wl.F16, 5242624),
    (4, 2, orc.HORING, wl.F16, 5242880), (2, 1, orc.RING, wl.F32, 2097152), (15, 5, orc.HRING, wl.BF16, 2097168),
    (2, 1, orc.RING, wl.BF16, 1218736), (2, 1, orc.RING, wl.BF16, 1218752), (2, 1, orc.RING, wl.F16, 1687488),
    (2, 1, orc.RING, wl.BF16, 1687504), (3, 1, orc.RING, wl.BF16, 1722216), (3, 1, orc.RING, wl.BF16, 1722240),
    (8, 2, orc.HORING, wl.BF16, 696416), (8, 2, orc.HORING, wl.BF16, 696448), (8, 4, orc.HRING, wl.F16, 1107120),
    (8, 1, orc.RING, wl.BF16, 1107200), (4, 2, orc.HORING, wl.F32, 696416), (4, 2, orc.HORING, wl.F32, 696432),
    (5, 1, orc.RING, wl.F32, 700000), (9, 1, orc.RING, wl.BF16, 720000)])
def test_a_range(paro, P, G, sched, dtype, ol):
    n = ol * G
    lay = orc.layout(P, G, [n])
    plan = paro.paro_plan(P, G, "III", [n], sched=sched, grad_dtype=[dtype])
    assert orc.state_range(lay, P - 1, "I")[1] == ol
    _last_rank(paro, plan, lay, P, dtype, sched, "III")


@pytest.mark.parametrize("route", ["table", "tensors"])
def test_one_chunk_with_exempt_tensors(paro, route, monkeypatch):
    """Where a tensor is exempt a step with pauses gives what it gives without weight decay, elsewhere what it gives without the mask."""
    if route == "tensors":
        monkeypatch.setenv("PARO_TILE_TABLE_MAX_TILES", "0")
    P, L, sizes = 2, 1500000, [700001, 999999, 3, 1299997]
    flags = [0, 1, 0, 1]
    exempt = torch.cat([torch.full((n,), bool(f)) for n, f in zip(sizes, flags)]).to(DEV)
    contrib = wl.chunk_contribs(P, L, 82, device=DEV)
    start = [t.to(DEV) for t in wl.master_state(L, 83)]

    def step(weight_decay, no_decay):
        plan = paro.paro_plan(P, 1, "IIG", sizes, no_decay=no_decay)
        p, m, v = (t.clone() for t in start)
        dst, ss = torch.zeros(P * L, dtype=torch.bfloat16, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)
        g = torch.empty(L, dtype=torch.float32, device=DEV)
        hp = hp_struct(paro, dict(hp_dict(P, max_norm=0.0), weight_decay=weight_decay), 3)
        paro.paro_step_fused(plan, 1, [c.data_ptr() for c in contrib], paro.PARO_CHUNK, hp, g.data_ptr(), ss.data_ptr(), p.data_ptr(),
                             m.data_ptr(), v.data_ptr(), dst.data_ptr(), stream())
        return p, m, v, dst[L:]

    got, decayed, plain = step(0.5, flags), step(0.5, None), step(0.0, None)
    assert not torch.equal(decayed[0], plain[0])
    own = exempt[L:]
    for g, d, o in zip(got, decayed, plain):
        assert torch.equal(g, torch.where(own, o, d))
