"""The sizes that the pulled gradient takes (csrc/internal.h, pull_fits), compiled
for the host: k_pull reads its entry lists at 32-bit word indexes, a batch of 64
words past the last, so every such index has to fit."""
import os
import subprocess

import pytest

from paper_2308_15020_amd import build

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "internal.h"
int main(int argc, char **argv)
{
    for (int i = 1; i + 3 < argc; i += 4)
        printf("%d\n", ffsat::pull_fits(atoll(argv[i]), atoll(argv[i + 1]), atoll(argv[i + 2]), atoi(argv[i + 3])) ? 1 : 0);
    printf("%d %d\n", ffsat::PULL_E[ffsat::PULL_LE3], ffsat::PULL_E[ffsat::PULL_LE7]);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pull_limits")
    src, exe = str(d / "limits.cpp"), str(d / "limits")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.check_call([build.HIPCC, "-std=c++17", f"--offload-arch={build.ARCH}", "-I", build.INCLUDE, "-I", build.CSRC,
                           "-x", "hip", src, "-o", exe], stderr=subprocess.DEVNULL)
    return exe


def test_every_index_fits(program):
    cases = []
    for E in (4, 8):
        most = (2**31 - 1 - 64) // E
        cases += [(10, 1, most, E, 1), (10, 1, most + 1, E, 0), (10, 1, 2**31 - 2, E, 0), (10, 1, 30, E, 1)]
    cases += [(2**19, 1023, 30, 4, 1), (2**19, 1024, 30, 4, 0)]
    args = [str(v) for c in cases for v in c[:4]]
    out = subprocess.check_output([program] + args, text=True).split()
    assert out[-2:] == ["4", "8"]
    assert [int(v) for v in out[:-2]] == [c[4] for c in cases]
    for n, B, lits, E, ok in cases:
        if ok:
            assert lits * E + 63 < 2**31 and n * B * 4 < 2**31
