"""The extension that reads the usual arguments of the device calls accepts, refuses and passes on what the ctypes
functions do.  Without a GPU every call ends in a refusal: which one tells what the library was handed."""
import ctypes
import inspect
import itertools
import os

import numpy as np
import pytest

import paper_2310_06003_amd as paro

HP = dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, grad_scale=0.25)


def outcome(call):
    try:
        return "returned", call()
    except paro.ParoError as e:
        return "refused", e.code, str(e)
    except Exception as e:
        return "raised", type(e)


FIELDS = [f for f, _ in paro.paro_adam_t._fields_]


@pytest.mark.parametrize("change", [
    {}, dict(step=7), dict(step=2**31 - 1), dict(step=2**31), dict(step=-1), dict(step=3.0), dict(step=True), dict(step=np.int64(4)),
    dict(lr=1), dict(lr=np.float32(0.1)), dict(lr=True), dict(lr="x"), dict(lr=None), dict(lr=1e300), dict(eps=float("nan")),
    dict(max_norm=1.0), dict(max_norm=2), dict(adamw=False), dict(adamw=0), dict(adamw=[1]), dict(skip_nonfinite=True),
    dict(skip_nonfinite=None), dict(unknown=1)])
def test_make_adam_gives_the_same_structure(change):
    def fields(f):
        kind = outcome(lambda: f(**{**HP, **change}))
        if kind[0] != "returned":
            return kind
        assert type(kind[1]) is paro.paro_adam_t
        return [(f, np.asarray(getattr(kind[1], f)).tobytes()) for f in FIELDS]
    assert fields(paro.make_adam) == fields(paro._through_ctypes["make_adam"])


def test_make_adam_is_keyword_only_and_complete():
    for f in (paro.make_adam, paro._through_ctypes["make_adam"]):
        with pytest.raises(TypeError):
            f(1e-4, **HP)
        for k in HP:
            with pytest.raises(TypeError):
                f(**{n: x for n, x in HP.items() if n != k})
    built = "".join(["l", "r"])                              # a name that the program made at run time
    assert paro.make_adam(**{**HP, built: 0.5}).lr == 0.5


def arguments(name, plan):
    """Arguments that the library refuses late: every pointer but the last one checked is in order."""
    hp, p = paro.make_adam(max_norm=1.0, **HP), 1 << 12
    c = [p] * 4
    return {
        "paro_reduce_shard": [plan, 1, c, paro.PARO_CHUNK, p, 8, 0],
        "paro_adam_shard": [plan, 1, hp, p, 8, p, p, p, p, 0],
        "paro_pack_params": [plan, 1, p, p, 0],
        "paro_step_fused": [plan, 1, c, paro.PARO_CHUNK, hp, p, 8, p, p, p, p, 0],
        "paro_step_fused_static": [plan, 1, c, hp, p, 8, p, p, p, p, 0],
        "paro_ring_hop": [plan, p, paro.PARO_F32, p, paro.PARO_BF16, p, -1, 0],
        "paro_collective_step": [plan, 1, -1, paro.PARO_AG, 9, 9, 9, c, 0],
    }[name]


NAMES = ["paro_reduce_shard", "paro_adam_shard", "paro_pack_params", "paro_step_fused", "paro_step_fused_static", "paro_ring_hop",
         "paro_collective_step"]
# in the place of one argument: misaligned and absent addresses, numbers out of range, other types
OTHERS = [0, 9, -1, None, 1 << 40, 1 << 63, 1 << 64, -(1 << 70), True, 1.5, "x", np.int64(16), ctypes.c_void_p(16), [], (), [16] * 4,
          (16,) * 4, [16, 9, 16, 16], [16, None, 16, 16], [np.int64(9)] * 4, [16] * 300, iter([16] * 4), object()]


@pytest.mark.skipif(__import__("torch").cuda.is_available(), reason="calls with made-up addresses are for machines without a GPU")
@pytest.mark.parametrize("name", NAMES)
def test_every_argument_is_read_as_ctypes_reads_it(name):
    plan = paro.paro_plan(4, 2, "IIG", [1 << 12])
    fast, slow = getattr(paro, name), paro._through_ctypes[name]
    good = arguments(name, plan)
    assert outcome(lambda: fast(*good)) == outcome(lambda: slow(*good))
    for k, x in itertools.product(range(len(good)), OTHERS):
        if isinstance(good[k], list) and isinstance(x, (list, tuple)) and len(x) < 4:
            continue                                         # fewer addresses than ranks: ctypes hands over an array too short
        args = good[:k] + [x] + good[k + 1:]
        if not isinstance(x, type(iter([]))):                # (an iterator has no second time)
            assert outcome(lambda: fast(*args)) == outcome(lambda: slow(*args)), (name, k, x)
    for n in range(len(good)):                               # defaults, and what has none
        assert outcome(lambda: fast(*good[:n])) == outcome(lambda: slow(*good[:n])), (name, n)
    names = list(inspect.signature(slow).parameters)
    assert names == list(inspect.signature(fast).parameters)
    assert outcome(lambda: fast(**dict(zip(names, good)))) == outcome(lambda: slow(**dict(zip(names, good))))
    assert outcome(lambda: fast(*good, 0)) == outcome(lambda: slow(*good, 0))
    tail = dict(zip(names[2:], good[2:]))
    assert outcome(lambda: fast(*good[:2], **tail)) == outcome(lambda: slow(*good[:2], **tail))


def test_a_list_too_short_for_its_plan_is_refused():
    plan = paro.paro_plan(4, 2, "IIG", [1 << 12])
    args = arguments("paro_reduce_shard", plan)
    with pytest.raises(paro.ParoError) as e:
        paro.paro_reduce_shard(*args[:2], [1 << 12] * 3, *args[3:])
    assert e.value.code == paro.PARO_EINVAL


def test_a_closed_plan_is_refused():
    plan = paro.paro_plan(4, 2, "IIG", [1 << 12])
    plan.__del__()
    with pytest.raises(paro.ParoError) as e:
        paro.paro_pack_params(plan, 1, 16, 16)
    assert e.value.code == paro.PARO_EINVAL


def test_another_interpreter_neither_trusts_nor_loads_this_ones_extension(monkeypatch):
    """The extension is compiled against one CPython's structures: in a tree built by this interpreter another one finds the
    build stale and the package refuses to import, until it is built again."""
    import __graft_entry__ as entry
    import importlib.util
    import sysconfig
    entry.ensure_built()
    assert not entry._lib_build_module().stale()
    here = sysconfig.get_config_var("EXT_SUFFIX")
    assert entry._lib_build_module().MARSHAL_SO == paro._marshal.__file__ and paro._marshal.__file__.endswith("_marshal" + here)
    real = sysconfig.get_config_var
    monkeypatch.setattr(sysconfig, "get_config_var", lambda k: ".cpython-399-other.so" if k == "EXT_SUFFIX" else real(k))
    other = entry._lib_build_module()
    assert other.stale() and other.source_hash() != other.built_hash()
    spec = importlib.util.spec_from_file_location("another_interpreters_package", paro.__file__,
                                                  submodule_search_locations=[os.path.dirname(paro.__file__)])
    with pytest.raises(ImportError, match="cpython-399-other"):
        spec.loader.exec_module(importlib.util.module_from_spec(spec))
