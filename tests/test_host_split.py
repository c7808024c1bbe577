"""How work is divided, on the CPU: the integer rules of csrc/ that the kernels and their host side share, compiled with g++."""
import ctypes
import os
import random
import subprocess

import pytest

import paper_2511_04477_amd as spqt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include <vector>
#include "split.hpp"
using namespace spqt;

// All shares of n things; 0 = right.  *corrected counts the quotients that the inverse gives one too large.
template <int WAVES>
static int check_shares(int n, int S, int *corrected) {
    const int parts = S * WAVES;
    const uint32_t inv = inverse_of(parts);
    if (WAVES > 1 && mul_hi((uint32_t)n, inv) != (uint32_t)(n / parts)) ++*corrected;
    for (int part = 0; part < parts; ++part) {
        const Share got = share_of<WAVES>(n, part, parts, inv);
        if (got.begin != (int)((int64_t)n * part / parts) || got.end != (int)((int64_t)n * (part + 1) / parts)) return 1;
    }
    return 0;
}

// Every workgroup of T block-rows once, the padding of the grid nowhere, block-rows that are not spread on one XCD; 0 = right.
template <int WAVES>
static int check_blocks(int T, int S) {
    const uint32_t inv = inverse_of(S * WAVES);
    std::vector<char> seen((size_t)T * S, 0);
    size_t n = 0;
    for (int i = 0, grid = grid_blocks(T, S); i < grid; ++i) {
        int t, s;
        if (!block_of<WAVES>((uint32_t)i, S, T, inv, t, s)) continue;
        if (t < 0 || t >= T || s < 0 || s >= S || seen[(size_t)t * S + s]++) return 1;
        if (!is_spread(t, T) && (t & 7) != (i & 7)) return 2;
        ++n;
    }
    return n == (size_t)T * S ? 0 : 3;
}

#define SPQT_FOR_WAVES(call) (waves == 1 ? call<1> : waves == 2 ? call<2> : waves == 4 ? call<4> : call<8>)
extern "C" {
int quantum(int batch, int compact) { return slice_quantum(batch, compact != 0); }
int shares(int waves, int n, int S, int *corrected) { return SPQT_FOR_WAVES(check_shares)(n, S, corrected); }
int blocks(int waves, int T, int S) { return SPQT_FOR_WAVES(check_blocks)(T, S); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2511_04477_amd", "csrc"), "-o", str(d / "rules.so"), str(d / "rules.cpp")], check=True)
    return ctypes.CDLL(str(d / "rules.so"))


def passes_of(begin, end, group, groups):
    """Passes over columns [begin, end) that are all kept, up to 64 of at most `groups` quantization groups each; one of at most 32
    columns counts 0.55 (the second half of its products is left out)."""
    n = 0.0
    while begin < end:
        to = min(end, begin + 64, (begin // group + groups) * group)
        n += 1.0 if to - begin > 32 else 0.55
        begin = to
    return n


@pytest.mark.parametrize("group", [128, 64])
@pytest.mark.parametrize("rows", [1, 2, 3, 4])
def test_one_launch_slices_take_no_more_passes_than_units(rules, rows, group):
    """Group layout, one launch, one range per slice: the longest slice takes no more passes than if slices were whole units of 64
    columns (up to half a pass more for 1 and 2 rows, where a slice that ends inside a unit gains more elsewhere than that)."""
    groups = {1: 4, 2: 2, 3: 1, 4: 1}[rows]
    q = rules.quantum(rows, 1)
    for M, K in [(512, 1024), (5120, 5120), (4096, 11008), (13678, 2816), (11001, 4224), (5321, 1920), (823, 1664), (2528, 7040),
                 (4096, 14336), (13824, 5120), (28672, 8192)]:
        splits, waves = spqt.spqt_default_cfg(M, K, rows, True)
        parts = splits * waves

        def longest(quantum):
            n = K // quantum
            return max(passes_of(n * p // parts * quantum, n * (p + 1) // parts * quantum, group, groups) for p in range(parts))
        assert longest(q) <= longest(64) + (0.55 if rows <= 2 else 0.0) + 1e-9, (M, K, parts, longest(q), longest(64))


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
def test_shares_are_those_of_exact_division(rules, waves):
    """n * part / parts rounded down, for every part; widths and kept counts from 0 to 2^24, where the inverse alone can be one off."""
    corrected = ctypes.c_int(0)
    edges = [e + d for e in (0, 128, 8192, 1 << 16, 1 << 20, 1 << 23, 1 << 24) for d in (-129, -2, -1, 0, 1, 63, 64)]
    random_n = random.Random(waves)
    for S in range(1, 65):
        for n in edges + [random_n.randrange(1 << 24) for _ in range(60)] + [(1 << 24) - random_n.randrange(1 << 12) for _ in range(60)]:
            if 0 <= n <= 1 << 24:
                assert rules.shares(waves, n, S, ctypes.byref(corrected)) == 0, (n, S)
    assert waves < 8 or corrected.value > 0      # the correction ran (only more than 256 parts need it)


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
def test_every_workgroup_has_one_place(rules, waves):
    """Up to the largest heights: 2^16 block-rows, 2^17 with the 8-bit layout's of 128 rows (4 wavefronts at most)."""
    highest = (1 << 16) if waves == 8 else 1 << 17
    for T in list(range(1, 42)) + [56, 112, 255, 256, 257, 1001]:
        for S in range(1, 65):
            assert rules.blocks(waves, T, S) == 0, (T, S)
    for T in (highest - 9, highest - 1, highest):
        for S in (1, 2, 3, 7, 12, 16, 31, 63, 64):
            assert rules.blocks(waves, T, S) == 0, (T, S)
