"""The vector loads of the tensor layout promise the compiler no more alignment than a gradient tensor has -
its elements' own: 2 bytes, or 4 for fp32 - and are still one instruction each.  Each loader is compiled
alone for gfx950, and its loads are read off the compiler's intermediate code and its assembly (no GPU)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DTYPES = {"bf16": ("PARO_BF16", 2, "dwordx2"), "f16": ("PARO_F16", 2, "dwordx2"), "f32": ("PARO_F32", 4, "dwordx4")}
LOADERS = {                                     # name: type, its members, vector loads, streaming
    "whole_nt": ("Tensor4Loader<{dt}, true>", "0, 0", 1, True),
    "whole": ("Tensor4Loader<{dt}, false>", "0, 0", 1, False),
    "pair_nt": ("Tensor8Loader<{dt}, true, 4>", "0, 0", 2, True),
    "pair": ("Tensor8Loader<{dt}, false, 8>", "0, 0", 2, False),
    "part": ("Part4Loader<{dt}>", "0, 0, a, b", 1, False),
}


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    where = tmp_path_factory.mktemp("loads")
    src = ['#include <hip/hip_runtime.h>', '#include "loaders.hpp"',
           "template <class Ld> __device__ void one(const Ld &ld, uintptr_t at, float *out) {",
           "    typename Ld::Raw r; ld.load(at, r);", "    float x[Ld::kElems]; ld.unpack(r, x);",
           "    for (int i = 0; i < Ld::kElems; ++i) out[threadIdx.x * Ld::kElems + i] = x[i];", "}"]
    for name, (loader, init, _count, _nt) in LOADERS.items():
        for d, (code, _align, _insn) in DTYPES.items():
            src.append(f'extern "C" __global__ void {name}_{d}(uintptr_t at, float *out, int a, int b) '
                       f"{{ one({loader.format(dt=code)}{{{init}}}, at, out); }}")
    hip = where / "loads.hip"
    hip.write_text("\n".join(src) + "\n")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2310_06003_amd", "csrc"), str(hip)]
    text = {}
    for kind, extra in (("ir", ["-emit-llvm"]), ("asm", [])):
        out = where / kind
        r = subprocess.run(cmd + extra + ["-o", str(out)], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
        text[kind] = out.read_text()
    return text


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("loader", list(LOADERS))
def test_alignment_of_the_vector_loads(compiled, loader, dtype):
    _code, align, insn = DTYPES[dtype]
    _type, _init, count, nt = LOADERS[loader]
    kernel = f"{loader}_{dtype}"
    ir = re.search(rf"^define [^\n]*@{kernel}\(.*?^}}", compiled["ir"], re.M | re.S).group(0)
    loads = re.findall(r"= load <\d+ x \w+>, ptr addrspace\(1\) [^,]+, align (\d+)(.*)", ir)
    assert [int(a) for a, _ in loads] == [align] * count
    assert all(("!nontemporal" in rest) == nt for _, rest in loads)
    asm = re.search(rf"^{kernel}:.*?s_endpgm", compiled["asm"], re.M | re.S).group(0)
    assert len(re.findall(rf"global_load_{insn}\b", asm)) == count
