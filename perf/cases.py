"""The work that users of the library have it do, as cases that can be timed and compared.

A case is a dict of plain values; `prepare` makes what a training program has in hand before the
call (gradient contributions, optimizer state, the plan), `run` makes ONE pass through the public
entry points, `exact` says in 64 bits what that pass returns.  Sizes are those of the workloads
that this repository is benchmarked and tested on (the 2^20-element list, the GPT-2-small-shaped
list, the ragged lists, the Llama-7B list) or lie between them.

Fields of a case
  call      "step"   paro_step_fused: reduce + (clip) + Adam + pack
            "static" paro_step_fused_static: the same without any allocation
            "split"  paro_reduce_shard, the cross-rank sum of squares, paro_adam_shard with pack
            "hop"    paro_ring_hop: one hop of a ring, or the accumulation of a micro-batch in place
            "gather" every rank's side of an all-gather, message by message (paro_collective_step)
  list      "flat" (one tensor of n elements), "gpt2", "llama" (n layers of width d), "ragged" (n
            tensors, sizes log-uniform in [1, 65536])
  P, G      ranks, ranks per group;  rank: the one whose share is worked on;  strategy: three letters
  layout    "chunk" or "tensors"
  dtype     of the contributions: "bf16", "f16", "f32", or "mixed" (a quarter of the tensors fp32)
  align     tensor layout: elements that every tensor's data is aligned to (128: separate
            allocations; 1: packed tight into one bucket)
  clip      global-norm clipping (a second sweep);  loss_scale: fp16 training, overflow skips the step
  no_decay  vectors are exempt from weight decay;  l2: classic L2 decay instead of AdamW
"""
import math

import numpy as np
import torch

import paper_2310_06003_amd as paro

DEV = "cuda:0"
CODE = {"bf16": paro.PARO_BF16, "f32": paro.PARO_F32, "f16": paro.PARO_F16}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}
SIZE = {"bf16": 2, "f32": 4, "f16": 2}
HP = dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
FIRST_STEP = 100        # mid-training: the bias corrections are no longer at their first values

STEP = dict(call="step", list="flat", n=1 << 20, d=0, P=4, G=2, rank=1, strategy="IIG", layout="chunk", dtype="bf16",
            align=128, clip=False, loss_scale=False, no_decay=False, l2=False)


def listed():
    return [
        # The smallest call: a 2^20-element model over 4 ranks, no clipping - one short kernel, latency.
        dict(STEP, name="tiny_step"),
        # A small odd-sized model, clipped, inside a loop that may not allocate (capture, serving):
        # several dependent short kernels.
        dict(STEP, name="small_static_clip", call="static", n=3_000_017, P=8, G=4, rank=6, clip=True),
        # GPT-2-small, data parallel with the optimizer state replicated (strategy NNN), fp16 gradients
        # with loss scaling and clipping: every rank updates all 8 chunks.
        dict(STEP, name="gpt2_replicated_f16", list="gpt2", P=8, G=8, rank=3, strategy="NNN", dtype="f16", clip=True,
             loss_scale=True),
        # GPT-2-small over 8 ranks, ZeRO-2 sharding, gradients handed over tensor by tensor, vectors exempt
        # from weight decay: the ordinary small training step.
        dict(STEP, name="gpt2_tensors_clip", list="gpt2", P=8, G=8, rank=5, strategy="NGG", layout="tensors", clip=True,
             no_decay=True),
        # 10 000 tensors of every size from 1 to 65536, a quarter with fp32 gradients: many small layers.
        dict(STEP, name="ragged_clip", list="ragged", n=10_000, P=8, G=4, rank=3, layout="tensors", dtype="mixed",
             clip=True),
        # The same law at a size that does not fit any cache, packed tight into flat gradient buckets
        # (arbitrary alignment), no clipping: the single sweep over tensors.
        dict(STEP, name="ragged_large_packed", list="ragged", n=160_000, P=8, G=4, rank=3, layout="tensors",
             dtype="mixed", align=1),
        # One GPU's share of Llama-7B over 16 ranks in groups of 8, PaRO-IIG, clipped: the flagship step.
        dict(STEP, name="llama7b_clip", n=6_738_415_616, P=16, G=8, rank=5, clip=True),
        # The same share from per-tensor gradients, no clipping.
        dict(STEP, name="llama7b_tensors", list="llama", n=32, d=4096, P=16, G=8, rank=5, layout="tensors"),
        # The same model over 64 ranks (8 groups of 8, PaRO-IGG), clipped: a wide fan-in.
        dict(STEP, name="llama7b_64ranks_clip", n=6_738_415_616, P=64, G=8, rank=21, strategy="IGG", clip=True),
        # MiCS sharding (state inside the group only, two chunks a rank), fp32 gradients, classic L2 decay,
        # through the split calls that a multi-GPU deployment puts its norm all-reduce between.
        dict(STEP, name="mics_split_f32", call="split", n=1_000_000_007, P=16, G=8, rank=11, strategy="III", dtype="f32",
             clip=True, l2=True),
        # A micro-batch's bf16 gradients accumulated into the fp32 shard of one rank of 8.
        dict(STEP, name="accumulate_bf16", call="hop", n=842_301_951),
        # The all-gather of GPT-2-small's parameters over 8 ranks in groups of 4, every message played.
        dict(STEP, name="gather_gpt2", call="gather", list="gpt2", P=8, G=4, strategy="IIG"),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    call = rng.choices(["step", "static", "split", "hop", "gather"], [55, 8, 20, 9, 8])[0]
    if call == "hop":
        return dict(STEP, call="hop", n=_log(rng, 1 << 14, 800_000_000), dtype=rng.choice(["bf16", "bf16", "f32", "f16"]))
    P = rng.choice([2, 4, 8, 8, 8, 16, 16, 16, 32, 64, 3, 6, 12, 24])
    G = rng.choice([g for g in range(1, P + 1) if P % g == 0 and (g > 1 or P < 5)])
    rank = rng.randrange(P)
    if call == "gather":
        P = min(P, 16)
        G = rng.choice([g for g in range(1, P + 1) if P % g == 0])
        return dict(STEP, call="gather", n=_log(rng, 1 << 16, 200_000_000 // P * 8 // P), P=P, G=G, rank=0)
    clip = rng.random() < 0.7
    base = dict(STEP, call=call, P=P, G=G, rank=rank, clip=clip, l2=rng.random() < 0.2)
    layout = "chunk" if call == "static" else rng.choice(["chunk", "tensors"])
    if layout == "tensors":
        base.update(layout="tensors", align=rng.choice([128, 128, 1]), no_decay=rng.random() < 0.4,
                    strategy=rng.choice(["IIG", "IGG", "NIG", "NGG", "GGG"]))
        kind = rng.choice(["gpt2", "llama", "ragged", "ragged"])
        if kind == "gpt2":
            return dict(base, list="gpt2", dtype=rng.choice(["bf16", "bf16", "f32", "f16"]))
        if kind == "llama":
            return dict(base, list="llama", n=_log(rng, 2, 24), d=256 * _log(rng, 2, 8), dtype=rng.choice(["bf16", "bf16", "f16"]))
        return dict(base, list="ragged", n=_log(rng, 200, 100_000), dtype=rng.choice(["mixed", "mixed", "bf16", "f32"]))
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
    strategy = rng.choice(["IIG", "IIG", "IGG", "NIG", "NGG", "GGG"]) if call == "static" else \
        rng.choice(["IIG", "IIG", "IGG", "NIG", "NGG", "GGG", "III", "III", "NNN"])
    # elements of the rank's update range; the contributions stay below the flagship step's
    rng_chunks = {"G": 1, "I": P // G, "N": P}[strategy[2]]
    most = min(400_000_000, 13_000_000_000 // (P * SIZE[dtype]))
    elems = _log(rng, min(most // 2, (1 << 14) * rng_chunks), most)
    n = max(1, elems * P // rng_chunks - rng.randrange(1, 64))
    return dict(base, n=n, dtype=dtype, strategy=strategy, loss_scale=dtype == "f16" and clip and call != "split")


# ------------------------------------------------------------------------------ shapes
def _sizes(case):
    kind, n = case["list"], case["n"]
    if kind == "flat":
        return [n]
    if kind == "gpt2":
        d = 768
        block = [d, d, 3 * d * d, d * d, d, d, 4 * d * d, 4 * d * d]
        return [50257 * d, 1024 * d] + block * 12 + [d, d]
    if kind == "llama":
        d = case["d"]
        f = d * 11008 // 4096
        layer = [d] + [d * d] * 4 + [d] + [d * f] * 3
        return [32000 * d] + layer * n + [d, 32000 * d]
    u = np.random.default_rng(5).random(n)                   # the list is the model's: not made from the seed
    return [int(x) for x in np.clip(np.floor(2.0 ** (16 * u)), 1, 65536)]


def _dtypes(case, count):
    if case["dtype"] != "mixed":
        return [case["dtype"]] * count
    u = np.random.default_rng(55).random(count)
    return ["f32" if x < 0.25 else "bf16" for x in u]


def _no_decay(case, sizes):
    return [1 if s <= 8192 else 0 for s in sizes] if case["no_decay"] else None


def _ranges(case, total):
    """L, own chunk's start, the update range and the parameter range (begin, length), in elements."""
    P, G = case["P"], case["G"]
    g = P // G
    L = -(-(-(-total // P)) // 8) * 8
    j, i = divmod(case["rank"], G)
    span = {"G": ((i * g + j) * L, L), "I": (i * g * L, g * L), "N": (0, P * L)}
    return L, (i * g + j) * L, span[case["strategy"][2]], span[case["strategy"][0]]


def _touched(sizes, begin, length):
    """Offsets of the tensors, and the first and the last of them that meet the range."""
    off = np.concatenate([[0], np.cumsum(np.asarray(sizes, dtype=np.int64))])
    meets = np.nonzero((off[:-1] < begin + length) & (off[1:] > begin) & (np.diff(off) > 0))[0]
    return off, int(meets[0]), int(meets[-1])


# ------------------------------------------------------------------------------ inputs
def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed((seed * 1_000_003 + salt * 7919 + 17) & 0x7FFFFFFFFFFF)


def _normal(n, seed, salt, scale, dtype):
    out = torch.empty(n, dtype=dtype, device=DEV)
    gen = _gen(seed, salt)
    for lo in range(0, n, 1 << 27):
        m = min(1 << 27, n - lo)
        z = torch.randn(m, generator=gen, device=DEV, dtype=torch.float32)
        out[lo:lo + m] = z.mul_(scale)
    return out


def _state(n, seed):
    """Master parameters and the two moments of a model in mid-training."""
    p = _normal(n, seed, 1, 0.02, torch.float32)
    m = _normal(n, seed, 2, 3e-5, torch.float32)
    v = _normal(n, seed, 3, 3e-5, torch.float32)
    return p, m, v.mul_(v).add_(1e-10)


def _grad_scale_of(case):
    return 1024.0 if case["loss_scale"] else 1.0


def _contribs(case, seed):
    """The ranks' gradients: in chunk layout one array over the update range each; in tensor layout one
    buffer per dtype each, and per tensor its dtype and first element in that buffer."""
    sizes = _sizes(case)
    total = sum(sizes)
    L, _own, (ob, ol), _par = _ranges(case, total)
    scale = 1e-3 * _grad_scale_of(case)
    if case["layout"] == "chunk":
        pad = max(0, ob + ol - total)
        out = []
        for q in range(case["P"]):
            x = _normal(ol, seed, 100 + q, scale, TORCH[case["dtype"]])
            if pad:
                x[max(0, ol - pad):] = 0
            out.append(x)
        return out, None, None
    dts = _dtypes(case, len(sizes))
    off, first, last = _touched(sizes, ob, ol)
    fill, start, a = {}, np.zeros(len(sizes), dtype=np.int64), case["align"]
    for t in range(first, last + 1):
        start[t] = fill.get(dts[t], 0)
        fill[dts[t]] = int(start[t]) + -(-sizes[t] // a) * a
    out = [{k: _normal(n, seed, 100 + q + 1000 * CODE[k], scale, TORCH[k]) for k, n in sorted(fill.items())}
           for q in range(case["P"])]
    return out, dts, start


def _gather_bytes(case):
    total = sum(_sizes(case))
    L = _ranges(case, total)[0]
    return L, case["P"] * L


def _schedule(plan, P):
    """Every rank's steps of the all-gather, in the order in which they are played."""
    steps = sorted({(m.phase, m.ring, m.step) for q in range(P) for m in paro.paro_schedule(plan, q, paro.PARO_AG)})
    return [(q, phase, ring, step) for (phase, ring, step) in steps for q in range(P)]


def prepare(case, seed):
    s = {"case": case, "stream": torch.cuda.current_stream().cuda_stream, "step": FIRST_STEP}
    if case["call"] == "hop":
        s["plan"] = paro.paro_plan(1, 1, "NNN", [case["n"]])
        s["acc"] = _normal(case["n"], seed, 4, 2e-3, torch.float32)
        s["local"] = _normal(case["n"], seed, 5, 1e-3, TORCH[case["dtype"]])
        return s
    sizes = _sizes(case)
    P, total = case["P"], sum(sizes)
    if case["call"] == "gather":
        s["plan"] = paro.paro_plan(P, case["G"], case["strategy"], sizes)
        L, n = _gather_bytes(case)
        s["bufs"] = []
        for q in range(P):
            b = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
            c = (q % case["G"]) * (P // case["G"]) + q // case["G"]
            b[c * L:(c + 1) * L] = _normal(L, seed, 6 + q, 0.02, torch.bfloat16)
            s["bufs"].append(b)
        s["ptrs"] = [b.data_ptr() for b in s["bufs"]]
        s["steps"] = _schedule(s["plan"], P)
        return s
    dts = _dtypes(case, len(sizes))
    f16 = case["dtype"] == "f16"
    plan = paro.paro_plan(P, case["G"], case["strategy"], sizes, grad_dtype=[CODE[k] for k in dts],
                          no_decay=_no_decay(case, sizes), pack_dtype=paro.PARO_F16 if f16 else paro.PARO_BF16)
    _L, _own, (ob, ol), (pb, pn) = _ranges(case, total)
    data, dts, start = _contribs(case, seed)
    if case["layout"] == "chunk":
        ptrs = [x.data_ptr() for x in data]
    else:
        _off, first, last = _touched(sizes, ob, ol)
        esize = np.asarray([SIZE[k] for k in dts], dtype=np.int64)
        tables = []
        for bufs in data:
            base = {k: b.data_ptr() for k, b in bufs.items()}
            spare = next(iter(base.values()))                # tensors outside the range: a valid address, never read
            at = np.full(len(sizes), spare, dtype=np.int64)
            use = slice(first, last + 1)
            at[use] = np.asarray([base[k] for k in dts[use]], dtype=np.int64) + start[use] * esize[use]
            tables.append(torch.from_numpy(at).to(DEV))
        s["tables"] = tables
        ptrs = [t.data_ptr() for t in tables]
    s["data"], s["ptrs"], s["plan"] = data, ptrs, plan
    s["p"], s["m"], s["v"] = _state(ol, seed)
    s["dst"] = torch.zeros(pn, dtype=torch.float16 if f16 else torch.bfloat16, device=DEV)
    if case["clip"] or case["call"] == "split":
        s["g"] = torch.zeros(ol, dtype=torch.float32, device=DEV)
        s["sumsq"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    s["hp"] = _hp(case)
    s["layout"] = paro.PARO_CHUNK if case["layout"] == "chunk" else paro.PARO_TENSORS
    return s


def _hp(case):
    return dict(HP, grad_scale=1.0 / (case["P"] * _grad_scale_of(case)), max_norm=1.0 if case["clip"] else 0.0,
                adamw=not case["l2"], skip_nonfinite=case["loss_scale"])


# ------------------------------------------------------------------------------ one pass
def run(s):
    case, st = s["case"], s["stream"]
    if case["call"] == "hop":
        acc = s["acc"].data_ptr()
        paro.paro_ring_hop(s["plan"], acc, paro.PARO_F32, s["local"].data_ptr(), CODE[case["dtype"]], acc, case["n"], st)
        return {"acc": s["acc"]}
    if case["call"] == "gather":
        for q, phase, ring, step in s["steps"]:
            paro.paro_collective_step(s["plan"], q, paro.PARO_SCHED_DEFAULT, paro.PARO_AG, phase, ring, step, s["ptrs"], st)
        return {"bufs": s["bufs"]}
    hp = paro.make_adam(step=s["step"], **s["hp"])
    s["step"] += 1
    p, m, v, dst = s["p"].data_ptr(), s["m"].data_ptr(), s["v"].data_ptr(), s["dst"].data_ptr()
    g, ss = (s["g"].data_ptr(), s["sumsq"].data_ptr()) if "g" in s else (0, 0)
    rank = case["rank"]
    if case["call"] == "split":
        paro.paro_reduce_shard(s["plan"], rank, s["ptrs"], s["layout"], g, ss, st)
        paro.paro_adam_shard(s["plan"], rank, hp, g, ss, p, m, v, dst, st)
    elif case["call"] == "static":
        paro.paro_step_fused_static(s["plan"], rank, s["ptrs"], hp, g, ss, p, m, v, dst, st)
    else:
        paro.paro_step_fused(s["plan"], rank, s["ptrs"], s["layout"], hp, g, ss, p, m, v, dst, st)
    return {k: s[k] for k in ("g", "sumsq", "p", "m", "v", "dst") if k in s}


# ------------------------------------------------------------------------------ what it costs at least
def work(case):
    n = case["n"]
    if case["call"] == "hop":
        return {"bytes": (8 + SIZE[case["dtype"]]) * n, "flops": n}
    sizes = _sizes(case)
    P = case["P"]
    if case["call"] == "gather":
        L, _n = _gather_bytes(case)
        return {"bytes": 4 * P * (P - 1) * L, "flops": 0}          # a rank receives P - 1 chunks: read and written
    total = sum(sizes)
    _L, _own, (ob, ol), _par = _ranges(case, total)
    if case["layout"] == "chunk":
        grads = P * ol * SIZE[case["dtype"]]
    else:
        off, first, last = _touched(sizes, ob, ol)
        dts = _dtypes(case, len(sizes))
        grads = sum(P * int(min(off[t + 1], ob + ol) - max(off[t], ob)) * SIZE[dts[t]] for t in range(first, last + 1))
    out = 4 if case["clip"] or case["call"] == "split" else 0
    return {"bytes": grads + (24 + 2 + out) * ol, "flops": (P + 20) * ol}


def tolerance(case):
    if case["call"] == "gather":
        return "exact"                                       # a copy
    if case["call"] == "hop":
        return {"rel": 1e-6}                                 # one fp32 add
    # The sums over ranks and of squares may be formed in another order (1e-7 in fp32), which moves a few packed
    # parameters by one unit in the last of their 8 bits.  Two evaluations whose step differs by 3e-7: 1.4e-5 and
    # 7e-3 (one unit) over the packed bf16, 4e-8 over the fp32 arrays.
    return {"rel": 6e-5, "max": 1e-2}


# ------------------------------------------------------------------------------ the same in 64 bits
def _sum_of_ranks(case, seed, sizes, ob, ol):
    data, dts, start = _contribs(case, seed)
    g = torch.zeros(ol, dtype=torch.float64, device=DEV)
    if case["layout"] == "chunk":
        while data:
            g += data.pop()
        return g
    off, first, last = _touched(sizes, ob, ol)
    for k in sorted(set(dts[first:last + 1])):
        mine = [t for t in range(first, last + 1) if dts[t] == k]
        lo = np.maximum(off[mine], ob)
        hi = np.minimum(off[[t + 1 for t in mine]], ob + ol)
        for a in range(0, len(mine), 4096):                  # where the tensors' elements lie, in the range and in the buffer
            where = [torch.arange(int(x - ob), int(y - ob), device=DEV) for x, y in zip(lo[a:a + 4096], hi[a:a + 4096])]
            count = torch.tensor([w.numel() for w in where], device=DEV)
            shift = torch.from_numpy(start[mine[a:a + 4096]] - (off[mine[a:a + 4096]] - ob)).to(DEV)
            to = torch.cat(where)
            frm = to + torch.repeat_interleave(shift, count)
            for bufs in data:
                g[to] += bufs[k][frm].double()
    return g


def exact(case, seed):
    if case["call"] == "hop":
        acc = _normal(case["n"], seed, 4, 2e-3, torch.float32).double()
        return {"acc": acc + _normal(case["n"], seed, 5, 1e-3, TORCH[case["dtype"]]).double()}
    if case["call"] == "gather":
        L, _n = _gather_bytes(case)
        P, G = case["P"], case["G"]
        chunks = [None] * P
        for q in range(P):
            chunks[(q % G) * (P // G) + q // G] = _normal(L, seed, 6 + q, 0.02, torch.bfloat16)
        return {"bufs": [torch.cat(chunks).double() for _ in range(P)] if 8 * P * P * L < 60e9 else [None] * P}
    sizes = _sizes(case)
    total = sum(sizes)
    L, own, (ob, ol), (pb, pn) = _ranges(case, total)
    g = _sum_of_ranks(case, seed, sizes, ob, ol)
    p, m, v = (x.double() for x in _state(ol, seed))
    hp = {k: float(np.float32(x)) if isinstance(x, float) else x for k, x in _hp(case).items()}
    sumsq = g[own - ob:own - ob + L].square().sum() if case["call"] == "split" else g.square().sum()
    scale = hp["grad_scale"]
    if case["clip"]:
        scale *= min(1.0, hp["max_norm"] / (hp["grad_scale"] * math.sqrt(float(sumsq)) + 1e-6))
    out = {}
    if case["clip"] or case["call"] == "split":
        out.update(g=g, sumsq=sumsq.reshape(1))
    decay = torch.full((ol,), hp["weight_decay"], dtype=torch.float64, device=DEV)
    exempt = _no_decay(case, sizes)
    if exempt:
        off, first, last = _touched(sizes, ob, ol)
        for t in range(first, last + 1):
            if exempt[t]:
                decay[max(0, int(off[t]) - ob):int(off[t + 1]) - ob] = 0
    d = g * scale
    if case["l2"]:
        d += decay * p
    m.mul_(hp["beta1"]).add_(d, alpha=1 - hp["beta1"])
    v.mul_(hp["beta2"]).addcmul_(d, d, value=1 - hp["beta2"])
    del d
    t = FIRST_STEP
    den = (v / (1 - hp["beta2"] ** t)).sqrt_().add_(hp["eps"])
    if not case["l2"]:
        p -= p * decay * hp["lr"]
    del decay
    p.addcdiv_(m, den, value=-hp["lr"] / (1 - hp["beta1"] ** t))
    del den
    dst = torch.zeros(pn, dtype=torch.float64, device=DEV)
    dst[ob - pb:ob - pb + ol] = p
    out.update(p=p, m=m, v=v, dst=dst)
    return out
