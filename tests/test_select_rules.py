"""The rule by which the selection of a row's best keys bounds them from below, against exact probabilities (no GPU)."""
import ctypes
import os
import subprocess

import pytest
from scipy.stats import hypergeom

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    (tmp / "rule.cpp").write_text('#include <math.h>\n#include "common.h"\nextern "C" void rule(int n, int k, int* out)\n'
                                  '{ const hr::TopkSample s = hr::topk_sample(n, k); out[0] = s.size; out[1] = s.want; out[2] = hr::kTopkCollect; }\n')
    so = str(tmp / "rule.so")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2507_09138_amd", "csrc"), str(tmp / "rule.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)

    def ask(n, k):
        out = (ctypes.c_int * 3)()
        lib.rule(n, k, out)
        return tuple(out)
    return ask


@pytest.mark.parametrize("n", [1, 63, 64, 256, 257, 300, 512, 513, 777, 1000, 1024])
def test_a_row_that_fits_the_buffer_never_misses_its_best(rule, n):
    """Whatever is wanted of it, up to all of its keys: the bound leaves out one of the best for less than one row in 10^9."""
    for k in range(1, min(n, 512) + 1):
        size, want, collect = rule(n, k)
        assert n <= collect
        if size:
            assert 1 <= want <= size and hypergeom.sf(want - 1, n, k - 1, size) < 1e-9, (n, k, size, want)


@pytest.mark.parametrize("n,most", [(1025, 512), (1500, 512), (2048, 512), (4096, 300), (4097, 512), (8192, 300), (16384, 200), (20000, 150), (32768, 40)])
def test_a_longer_row_collects_enough_and_not_too_many(rule, n, most):
    """What the rule's comment states: at most one row in 10^5 on either side."""
    for k in range(1, most + 1):
        size, want, collect = rule(n, k)
        assert 2 <= want <= size <= n
        assert hypergeom.sf(want - 1, n, k - 1, size) < 1e-5, (n, k, size, want)
        assert hypergeom.cdf(want - 1, n, collect, size) < 2e-5, (n, k, size, want)


def test_the_bound_is_a_sampled_key_for_every_size(rule):
    for n in [1025, 4096, 4097, 65536, 1 << 20, (1 << 24) - 1]:
        for k in (1, 2, 10, 128, 511, 512):
            size, want, _ = rule(n, k)
            assert 2 <= want <= size <= 1024
