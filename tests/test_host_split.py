"""How work is divided, on the CPU: the integer rules of csrc/ that the kernels and their host side share, compiled with g++."""
import ctypes
import os
import subprocess

import pytest

import paper_2511_04477_amd as spqt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "spqt_internal.h"
extern "C" int quantum(int batch, int compact) { return spqt::slice_quantum(batch, compact != 0); }
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
