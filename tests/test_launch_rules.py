"""Which kernels a call launches, with how many blocks and how much unused LDS (what thins out their waves), on the CPU: the
built library runs against a runtime of a few lines that only writes down what it is asked to launch.  Every pointer is made up."""
import os
import subprocess

import pytest

import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
M = 1 << 20
MAIN = r"""
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
#include "paro.h"

struct dim3 { uint32_t x, y, z; };
static dim3 grid_, block_;
static size_t lds_;
static std::map<const void *, std::string> &kernels() { static std::map<const void *, std::string> k; return k; }
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) {
    int status;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string n = status == 0 ? plain : name;
    std::free(plain);
    for (size_t at; (at = n.find("(anonymous namespace)::")) != std::string::npos;) n.erase(at, 23);
    kernels()[host] = n.rfind("void ", 0) == 0 ? n.substr(5) : n;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *) { grid_ = grid; block_ = block; lds_ = lds; return 0; }
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **st) { *grid = grid_; *block = block_; *lds = lds_; *st = nullptr; return 0; }
int hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t lds, void *) {
    std::printf("%s\t%u\t%zu\t%lld\n", kernels()[f].c_str(), grid.x, lds, (long long)*(const uintptr_t *)args[1]);
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 160 * 1024; return 0; }
int hipMalloc(void **p, size_t n) { return (*p = std::malloc(n)) ? 0 : 2; }
int hipFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *to, const void *from, size_t n, int) { std::memcpy(to, from, n); return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "?"; }
int hipGetSymbolAddress(void **p, const void *) { static double one; *p = &one; return 0; }
}

int main(int argc, char **) {
    if (argc > 1) {
        for (const auto &k : kernels()) std::printf("%s\n", k.second.c_str());
        return 0;
    }
    char call[16], letters[8];
    int P, G, rank, dtype, layout, clip, T;
    while (std::scanf("%15s %d %d %7s %d %d %d %d %d", call, &P, &G, letters, &rank, &dtype, &layout, &clip, &T) == 9) {
        std::vector<int64_t> sizes((size_t)T);
        std::vector<uint8_t> exempt((size_t)T), types((size_t)T, (uint8_t)dtype);
        for (auto &s : sizes) { long x; if (std::scanf("%ld", &x) != 1) return 1; s = x; }
        for (auto &e : exempt) { int x; if (std::scanf("%d", &x) != 1) return 1; e = (uint8_t)x; }
        const paro_plan_opts_t o = {PARO_SCHED_DEFAULT, 0, types.data(), exempt.data(), PARO_BF16, 0};
        paro_plan_t *pl = nullptr;
        if (paro_plan(P, G, letters, sizes.data(), T, &o, &pl) != PARO_OK) return 2;
        const auto at = [](int i) { return reinterpret_cast<void *>((uintptr_t)(i + 1) << 40); };
        std::vector<const void *> contrib;
        for (int q = 0; q < P; ++q) contrib.push_back(at(q));
        const paro_adam_t hp = {1e-4f, 0.9f, 0.999f, 1e-8f, 0.01f, 1.0f / P, clip ? 1.0f : 0.0f, 3, 1, 0};
        float *g = (float *)at(300), *p = (float *)at(301), *m = (float *)at(302), *v = (float *)at(303);
        double *ss = (double *)at(304);
        uint16_t *dst = (uint16_t *)at(305);
        int rc;
        if (!std::strcmp(call, "step")) rc = paro_step_fused(pl, rank, contrib.data(), layout, &hp, g, ss, p, m, v, dst, nullptr);
        else if (!std::strcmp(call, "reduce")) rc = paro_reduce_shard(pl, rank, contrib.data(), layout, g, ss, nullptr);
        else rc = paro_adam_shard(pl, rank, &hp, g, ss, p, m, v, dst, nullptr);
        if (rc != PARO_OK) { std::printf("%s\n", paro_last_error()); return 3; }
        std::printf("end\n");
        paro_plan_destroy(pl);
    }
    return 0;
}
"""


class Launch:
    def __init__(self, line):
        name, grid, lds, second = line.split("\t")
        self.name, self.args = name[:name.index("(")], name[name.index("("):]
        self.kernel, self.grid, self.lds, self.second = self.name.split("<")[0], int(grid), int(lds), int(second)

    @property
    def flags(self):
        return [x.strip() for x in self.name[self.name.index("<") + 1:-1].split(",")]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from __graft_entry__ import ensure_built
    ensure_built()
    where = tmp_path_factory.mktemp("launches")
    (where / "main.cpp").write_text(MAIN)
    lib = os.path.join(ROOT, "paper_2310_06003_amd")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), str(where / "main.cpp"), "-o", str(where / "launches"),
                        os.path.join(lib, "libparo.so"), "-Wl,-rpath," + lib, "-Wl,--allow-shlib-undefined", "-rdynamic"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return str(where / "launches")


@pytest.fixture(scope="module")
def launches(program):
    def ask(call, P, G, strategy, rank, dtype, layout, clip, sizes, exempt=None):
        line = f"{call} {P} {G} {strategy} {rank} {dtype} {layout} {int(clip)} {len(sizes)} " + \
            " ".join(map(str, list(sizes) + [int(x) for x in exempt or [0] * len(sizes)]))
        r = subprocess.run([program], input=line, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout[-500:] + r.stderr
        lines = r.stdout.splitlines()
        assert lines[-1] == "end"
        return [Launch(x) for x in lines[:-1]]
    return ask


@pytest.fixture(scope="module")
def kernels(program):
    return subprocess.run([program, "kernels"], capture_output=True, text=True, check=True).stdout.splitlines()


def test_the_parts_of_a_clipped_step(launches):
    got = launches("step", 8, 4, "IIG", 3, wl.BF16, 0, True, [8 * M])
    assert [x.kernel for x in got] == ["k_reduce4", "k_finalize", "k_adam4"] and [x.grid for x in got] == [4096, 8, 4096]


def test_launches_without_write_windows_do_not_carry_them(kernels):
    """Not even as an empty argument: what a small step pays for is the launch."""
    assert len(kernels) > 100
    assert [k for k in kernels if "Window" in k] == []


def test_no_single_sweep_with_windows_for_few_two_byte_contributions(kernels):
    """A launch has them from 64 bytes of contributions an element on, over a range of several chunks from 28 two-byte ones on: never with
    the table of 16 pointers, unless they are of fp32."""
    sweeps = [Launch(k + "\t0\t0\t0") for k in kernels if k.startswith(("k_fused4<false", "k_fused4r<"))]
    kinds = {(x.flags[1] if x.kernel == "k_fused4" else x.flags[0], x.flags[-3], x.flags[-1]) for x in sweeps}
    f32 = str(wl.F32)
    assert kinds == {(str(d), n, held) for d in (wl.BF16, wl.F16, wl.F32) for n in ("16", "256") for held in ("false", "true")
                     if held == "false" or n == "256" or str(d) == f32}


@pytest.mark.parametrize("P,G,strategy,dtype,L,held", [
    (32, 8, "IGG", wl.BF16, 26 * M, True), (32, 8, "IGG", wl.F16, 26 * M - 8, False), (32, 8, "IGG", wl.BF16, 19 * M, False),
    (33, 11, "IGG", wl.BF16, 13 * M, True), (40, 8, "IGG", wl.BF16, 7 * M, True), (31, 31, "IGG", wl.BF16, 40 * M, False), (16, 8, "IGG", wl.F32, 13 * M, True),
    (15, 5, "IGG", wl.F32, 40 * M, False), (28, 14, "III", wl.F16, 8 * M, True), (27, 9, "III", wl.F16, 8 * M, False),
    (16, 8, "III", wl.F32, 8 * M, True), (16, 8, "III", wl.BF16, 40 * M, False)])
def test_single_sweeps_with_windows(launches, P, G, strategy, dtype, L, held):
    assert [x.flags[-1] for x in launches("step", P, G, strategy, 1, dtype, 0, False, [P * L])] == [str(held).lower()]


@pytest.mark.parametrize("call,layout", [("step", 0), ("step", 1), ("adam", 0)])
def test_sweep_2_with_exempt_tensors_goes_from_the_start(launches, call, layout):
    got = [x for x in launches(call, 4, 2, "III", 1, wl.BF16, layout, True, [20 * M, 1000, 90 * M], [0, 1, 0]) if x.kernel == "k_adam4"]
    assert len(got) == 2 and got[0].second < got[1].second          # one launch a chunk: where its gradient begins


# Over one chunk of two-byte contributions: up to 16 ranks 49 152 blocks times ranks, up to 31 ranks 3840 blocks, then 4096, as with fp32 ones.
@pytest.mark.parametrize("P,G,strategy,dtype,blocks,all_waves", [
    (12, 4, "IGG", wl.BF16, 4096, True), (14, 7, "IGG", wl.F16, 3510, True), (14, 7, "IGG", wl.BF16, 3511, False), (16, 8, "IGG", wl.BF16, 3072, True),
    (16, 8, "IGG", wl.BF16, 3073, False), (17, 17, "IGG", wl.BF16, 3840, True), (31, 31, "IGG", wl.F16, 3841, False), (32, 8, "IGG", wl.BF16, 4096, True),
    (64, 8, "IGG", wl.BF16, 4097, False), (65, 13, "IGG", wl.BF16, 1000, False), (11, 11, "IGG", wl.BF16, 4000, False), (16, 8, "IGG", wl.F32, 4096, True),
    (16, 8, "III", wl.BF16, 4096, True), (12, 6, "III", wl.BF16, 1000, False), (24, 12, "III", wl.F32, 2048, True), (128, 64, "III", wl.BF16, 4096, True)])
def test_small_single_sweeps_with_all_waves(launches, P, G, strategy, dtype, blocks, all_waves):
    got, = launches("step", P, G, strategy, 1, dtype, 0, False, [P * blocks * 256])
    assert got.kernel in ("k_fused4", "k_fused4r") and (got.lds == 0) == all_waves


# Sweep 1 over per-tensor gradients runs all waves that fit with 48 ranks and more from 16 384 blocks on; large chunks (131 072 blocks) of fp32
# gradients only with 56 and more, in few large tensors.
@pytest.mark.parametrize("P,G,dtype,blocks,small,all_waves", [
    (48, 8, wl.BF16, 16384, False, True), (48, 8, wl.BF16, 16383, False, False), (47, 47, wl.BF16, 16384, False, False), (48, 8, wl.F32, 131071, False, True),
    (48, 8, wl.F32, 131072, False, False), (55, 11, wl.F32, 131072, False, False), (56, 8, wl.F32, 131072, False, True),
    (64, 8, wl.F32, 131072, True, False), (64, 8, wl.BF16, 131072, True, True)])
def test_sweep_1_over_tensors_of_many_ranks(launches, P, G, dtype, blocks, small, all_waves):
    L = blocks * 256
    own = [100_000] * (L // 100_000) + [L % 100_000] if small else [L]      # the first rank's chunk; every other is one tensor
    got = launches("reduce", P, G, "IGG", 0, dtype, 1, True, own + [L] * (P - 1))
    assert got[0].kernel == "k_reduce4t" and (got[0].lds == 0) == all_waves


# A chunk's blocks are counted with the one more that it may straddle, and in eights.
@pytest.mark.parametrize("P,G,dtype,blocks,one_by_one", [
    (4, 2, wl.BF16, 65536, True), (4, 2, wl.BF16, 65528, False), (8, 4, wl.BF16, 262144, False), (12, 6, wl.BF16, 131072, True), (12, 6, wl.F16, 131064, False),
    (32, 16, wl.F16, 65536, False), (64, 32, wl.BF16, 32768, False), (99, 33, wl.BF16, 131072, True), (100, 50, wl.BF16, 131072, False),
    (4, 2, wl.F32, 131072, False), (8, 4, wl.F32, 131072, True), (11, 1, wl.F32, 131072, True), (8, 4, wl.F32, 131064, False),
    (12, 6, wl.F32, 131072, False), (16, 8, wl.F32, 65536, False)])
def test_ranges_that_are_swept_chunk_by_chunk(launches, P, G, dtype, blocks, one_by_one):
    got = [x.kernel for x in launches("step", P, G, "III", 0, dtype, 0, True, [P * (blocks - 8) * 256]) if x.kernel.startswith("k_reduce")]
    assert got == ["k_reduce4"] * (P // G) if one_by_one else got == ["k_reduce4r"]
