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
void stats_chunks(int64_t tiles, int items, int n_cu, int most, double unit_tiles, int *nc, int *ct) {
    cb::choose_stats_chunks(tiles, items, n_cu, most, unit_tiles, nc, ct);
}
void even_chunks(int64_t tiles, int items, int n_cu, int *nc, int *ct) {
    cb::choose_chunks(tiles, items, n_cu, 0, nc, ct);
}
int most_chunks(int64_t tiles, int items, int n_cu) { return cb::most_stats_chunks(tiles, items, n_cu); }
double stats_error2(int64_t tiles, int64_t ct) { return cb::stats_error2(tiles, ct); }
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
    ip = ctypes.POINTER(ctypes.c_int)
    lib.stats_chunks.argtypes = [i64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_double, ip, ip]
    lib.even_chunks.argtypes = [i64, ctypes.c_int, ctypes.c_int, ip, ip]
    lib.most_chunks.argtypes = [i64, ctypes.c_int, ctypes.c_int]
    lib.stats_error2.argtypes, lib.stats_error2.restype = [i64, i64], ctypes.c_double
    return lib


def _chunks(f, *args):
    nc, ct = ctypes.c_int(-1), ctypes.c_int(-1)
    f(*args, ctypes.byref(nc), ctypes.byref(ct))
    return nc.value, ct.value


# Chunks of the moments: they cover the tiles, an fp32 sum runs over at most 2048 tiles, chunks other than eight units per
# compute unit are longer and leave at most three quarters of their squared error, and a plan's workspace holds them for every call of up to its tiles.
@pytest.mark.parametrize("unit_tiles", [5.3, 10.0, 35.3])
@pytest.mark.parametrize("items", [1, 2, 6, 64, 76, 160, 161, 320, 512, 640, 2049, 5120])
def test_stats_chunks_hold_their_bounds(rules, items, unit_tiles):
    for limit in [1, 31, 33, 500, 1030, 6400, 38936, 70000]:
        most = rules.most_chunks(limit, items, 256)
        sizes = sorted({t for k in range(1, 60) for t in (limit * k // 59, limit // k)} | {1, limit}) if limit > 600 else \
            range(1, limit + 1)
        for tiles in sizes:
            if tiles < 1:
                continue
            nc, ct = _chunks(rules.stats_chunks, tiles, items, 256, most, unit_tiles)
            n0, ct0 = _chunks(rules.even_chunks, tiles, items, 256)
            assert 1 <= nc <= most and (nc - 1) * ct < tiles <= nc * ct and ct <= 2048, (tiles, limit, nc, ct)
            assert ct >= ct0 and (ct == ct0 or rules.stats_error2(tiles, ct) <= 0.75 * rules.stats_error2(tiles, ct0)), \
                (tiles, limit, nc, ct, ct0)


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
