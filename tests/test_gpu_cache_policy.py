"""Results that the memory-side cache is to keep - a small gradient array, a small model's state, a ring's message - are
stored another way than large ones.  Sizes at both sides of every limit, against the oracle bit for bit."""
import pytest
import torch

import oracle as orc
import workloads as wl
from harness import DEV, hp_dict, np_of, run_rank, stream

pytestmark = pytest.mark.gpu

M = 1 << 20


@pytest.mark.parametrize("P,strategy,L,dtype", [
    (2, "NNG", M, wl.BF16), (2, "NNG", M + 8, wl.BF16), (2, "NNG", 4 * M, wl.F16), (2, "NNG", 4 * M + 8, wl.BF16),
    (2, "NNG", 16 * M, wl.BF16), (2, "NNG", 16 * M + 8, wl.BF16), (2, "NNN", 8 * M, wl.BF16), (2, "NNN", 8 * M + 8, wl.BF16),
    (16, "NNG", 6 * M, wl.BF16), (16, "NNG", 6 * M + 8, wl.BF16), (24, "NNG", M, wl.BF16), (24, "NNG", M + 8, wl.BF16),
    (8, "NNG", 8 * M, wl.F32), (8, "NNG", 8 * M + 8, wl.F32)])
def test_steps_at_the_limits(paro, P, strategy, L, dtype):
    lay = orc.layout(P, 1, [P * L])
    pl = paro.paro_plan(P, 1, strategy, [P * L], sched=orc.RING, grad_dtype=[dtype])
    rank = P - 1
    ob, ol = orc.state_range(lay, rank, strategy[2])
    dev = wl.chunk_contribs(P, ol, 70 + P, dtype=dtype, device=DEV)
    padded = [_Shifted(t, ob) for t in dev]
    state = [_Shifted(np_of(t), ob) for t in wl.master_state(ol, 71)]
    host = [_Shifted(np_of(t), ob) for t in dev]
    for max_norm in (0.0, 0.01):
        run_rank(paro, pl, lay, strategy, orc.RING, rank, padded, host, state, hp_dict(P, max_norm=max_norm), 5,
                 check_unfused=max_norm > 0)


class _Shifted:
    """An array over the rank's update range, indexed as one over the whole padded buffer."""

    def __init__(self, data, begin):
        self.data, self.begin = data, begin

    def __getitem__(self, s):
        return self.data[s.start - self.begin:s.stop - self.begin]


@pytest.mark.parametrize("n", [12 * M - 3, 12 * M, 12 * M + 1])
def test_hops_at_the_limit(paro, n):
    pl = paro.paro_plan(1, 1, "NNN", [64])
    a, b = torch.randn(n, device=DEV), torch.randn(n, device=DEV).bfloat16()
    want = a + b.float()
    paro.paro_ring_hop(pl, a.data_ptr(), wl.F32, b.data_ptr(), wl.BF16, a.data_ptr(), n, stream())
    assert torch.equal(a, want)


@pytest.mark.parametrize("L", [24 * M, 24 * M + 8])
def test_all_gather_messages_at_the_limit(paro, L):
    pl = paro.paro_plan(2, 1, "IIG", [2 * L])
    bufs = [torch.randn(2 * L, device=DEV).bfloat16() for _ in range(2)]
    want = torch.cat([bufs[r][c * L:(c + 1) * L] for c in range(2) for r in [paro.paro_owner_of_chunk(pl, c)]])
    for m in paro.paro_schedule(pl, 0, paro.PARO_AG):
        for q in range(2):
            paro.paro_collective_step(pl, q, paro.PARO_SCHED_DEFAULT, paro.PARO_AG, m.phase, m.ring, m.step,
                                      [b.data_ptr() for b in bufs], stream())
    assert all(torch.equal(b, want) for b in bufs)
