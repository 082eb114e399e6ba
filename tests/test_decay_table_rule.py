"""The weight-decay table of a chunk (host code, no GPU) against a count over every element, and the time it takes to make:
the program waits for it in the first call with a plan."""
import os
import subprocess

import numpy as np
import pytest

import oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BLOCK = 256
ALL, NONE, BITS = 0, 1, 2
MAIN = r"""
#include <chrono>
#include <cstdio>
#include <cstring>
#include "plan.hpp"
extern "C" void paro_plan_destroy(paro_plan_t *pl) { delete pl; }
using clk = std::chrono::steady_clock;
// the flags element by element
static void by_element(const paro_plan_t *pl, int64_t c, std::vector<uint8_t> *flags) {
    flags->assign((size_t)pl->L, 1);
    paro::for_each_tile(pl, c, [&](int64_t, int64_t f0, int64_t f1, int64_t k) {
        for (; k < (int64_t)pl->nz_tensor.size() && pl->nz_off[(size_t)k] < f1; ++k)
            for (int64_t x = std::max(pl->nz_off[(size_t)k], f0), e = std::min(pl->nz_off[(size_t)k + 1], f1); x < e; ++x)
                (*flags)[(size_t)(x - c * pl->L)] = !pl->no_decay[(size_t)pl->nz_tensor[(size_t)k]];
    });
}
template <class F>
static double least(F f) {
    double best = 1e9;
    for (int r = 0; r < 15; ++r) {
        const auto t = clk::now();
        f();
        best = std::min(best, std::chrono::duration<double>(clk::now() - t).count());
    }
    return best;
}
int main(int argc, char **argv) {
    int P; long T, x;
    while (std::scanf("%d %ld", &P, &T) == 2) {
        std::vector<int64_t> sizes;
        std::vector<uint8_t> nd, flags;
        std::vector<uint32_t> tab;
        for (long t = 0; t < T; ++t) { if (std::scanf("%ld", &x) != 1) return 1; sizes.push_back(x); }
        for (long t = 0; t < T; ++t) { if (std::scanf("%ld", &x) != 1) return 1; nd.push_back((uint8_t)x); }
        paro_plan_opts_t o = {PARO_SCHED_DEFAULT, 0, nullptr, nd.data(), PARO_BF16, 0};
        paro_plan_t *pl = nullptr;
        if (paro_plan(P, 1, "GGG", sizes.data(), T, &o, &pl) != PARO_OK) return 2;
        if (argc > 1) {
            std::printf("%g %g\n", least([&] { paro::list_decays(pl, 0, &tab); }), least([&] { by_element(pl, 0, &flags); }));
        } else {
            for (int c = 0; c < P; ++c) {
                paro::list_decays(pl, c, &tab);
                for (uint32_t w : tab) std::printf("%u ", w);
                std::printf("\n");
            }
        }
        paro_plan_destroy(pl);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    where = tmp_path_factory.mktemp("decay")
    (where / "main.cpp").write_text(MAIN)
    csrc = os.path.join(ROOT, "paper_2310_06003_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O3", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(csrc, "plan.cpp"), str(where / "main.cpp"), "-o", str(where / "rule"), "-lpthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def call(P, sizes, flags, *args):
        text = f"{P} {len(sizes)} " + " ".join(map(str, sizes)) + " " + " ".join(map(str, flags))
        r = subprocess.run([str(where / "rule"), *args], input=text, capture_output=True, text=True)
        assert r.returncode == 0
        return [[float(x) if args else int(x) for x in line.split()] for line in r.stdout.splitlines()]
    return call


def read(table, tiles, n):
    """What the kernels make of a table: a flag for each of the chunk's n elements."""
    out = []
    for entry in table[:tiles]:
        if entry < BITS:
            out += [entry == ALL] * BLOCK
        else:
            words = table[entry - BITS:entry - BITS + BLOCK // 32]
            assert entry - BITS >= tiles and len(words) == BLOCK // 32
            out += [bool(w >> b & 1) for w in words for b in range(32)]
    return np.array(out[:n])


def random_lists():
    rng = np.random.default_rng(90)
    for k in range(40):
        most = int(rng.choice([3, 40, 300, 2000]))
        sizes = [int(x) for x in rng.integers(0, most, int(rng.integers(1, 60)))] + [int(rng.integers(1, 3000))]
        yield sizes, [int(x) for x in rng.random(len(sizes)) < rng.choice([0.1, 0.5, 0.9])]


LISTS = [([256, 256, 255, 257, 512, 1, 255, 768], [0, 1, 1, 0, 1, 0, 1, 0]), ([32] * 40, [0, 1] * 20), ([31, 33, 1, 63, 64, 65], [1, 0] * 3),
         ([100, 156, 0, 256, 128, 64, 64, 300], [1, 1, 0, 0, 1, 1, 1, 0]), ([1000, 501], [1, 1]), ([1000, 501], [0, 0]),
         ([1] * 512 + [40], [int(i % 3 == 0) for i in range(513)]), ([5], [1])] + list(random_lists())


@pytest.mark.parametrize("P", [1, 2, 5])
def test_the_table_says_what_every_element_does(ask, P):
    for sizes, flags in LISTS:
        L = orc.layout(P, 1, sizes).L
        takes = np.concatenate([np.repeat(np.array(flags) == 0, sizes), np.full(P * L - sum(sizes), True)])
        tiles = -(-L // BLOCK)
        for c, table in enumerate(ask(P, sizes, flags)):
            want = takes[c * L:(c + 1) * L]
            np.testing.assert_array_equal(read(table, tiles, L), want)
            for i, entry in enumerate(table[:tiles]):                # words only where a tile needs them
                part = want[i * BLOCK:(i + 1) * BLOCK]
                assert (entry >= BITS) == (part.any() and not part.all())


def test_the_table_is_made_faster_than_element_by_element(ask):
    """Tensors of some 100 elements, every second exempt: each tile is mixed.  The bound is loose: made word by word the
    table takes a tenth of the time, bit by bit (as it once was) about as long as the elements."""
    sizes = [int(x) for x in np.random.default_rng(91).integers(60, 140, 60_000)]
    (made, elements), = ask(1, sizes, [k & 1 for k in range(len(sizes))], "time")
    assert made < 0.5 * elements, (made, elements)
