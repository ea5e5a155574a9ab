"""Host checks (no GPU) of the rules that cut a call's work into workgroups."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_00891_amd", "csrc")
SOURCE = """
#include "cb_rules.h"
extern "C" {
int64_t apply_sub_blocks(int64_t sub, int64_t groups, int64_t n_cu, int64_t resident, int64_t bytes) {
    return cb::choose_apply_sub_blocks(sub, groups, n_cu, resident, bytes);
}
double apply_cost(int64_t sub, int64_t per, int64_t groups, int64_t n_cu, int64_t resident, double rate) {
    return cb::apply_cost(sub, per, groups, n_cu, resident, rate);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    so = str(d / "librules.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "rules.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    i64 = ctypes.c_int64
    lib.apply_sub_blocks.argtypes, lib.apply_sub_blocks.restype = [i64] * 5, i64
    lib.apply_cost.argtypes, lib.apply_cost.restype = [i64] * 5 + [ctypes.c_double], ctypes.c_double
    return lib


# Application tiles: the chosen one costs at most 10% more than the best of all, and at most 5% more than tiles of at least
# 256 tokens at about 16 workgroups per compute unit, from one source block to hundreds and up to 262,144 tokens.
@pytest.mark.parametrize("resident,bytes_per", [(1, 16384), (1, 24576), (2, 10240), (3, 8192), (3, 12288)])
@pytest.mark.parametrize("groups", [1, 2, 3, 4, 7, 16, 40, 256, 260, 320, 640])
def test_apply_tiles_near_the_cheapest(rules, groups, resident, bytes_per):
    rate = min(1.0, bytes_per / 10240)
    for sub in [1, 2, 7, 25, 64, 100, 255, 256, 257, 512, 777, 1024, 2048, 4096, 8192]:
        per = rules.apply_sub_blocks(sub, groups, 256, resident, bytes_per)
        assert 1 <= per <= min(sub, 256)
        cost = lambda p: rules.apply_cost(sub, p, groups, 256, resident, rate)
        best = min(cost(p) for p in range(1, min(sub, 256) + 1))
        t = max((32 * sub * groups + 16 * 256 - 1) // (16 * 256), 256)
        wide = min((min(t, 8192) + 31) // 32, sub)
        assert cost(per) <= 1.1 * best, (sub, groups, per)
        assert cost(per) <= 1.05 * cost(wide), (sub, groups, per)
