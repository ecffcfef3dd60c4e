"""The order in which calls without an index deal their items to the XCDs, on
the CPU: the functions of csrc/internal.h compiled for the host."""
import ctypes
import os
import subprocess

import pytest

from paper_2607_09385_amd import build

SOURCE = """
#include "internal.h"
extern "C" {
int items(int units, int nQB, int range, int x) { return steel::coord_items(units, nQB, range, x); }
void order(int units, int nQB, int range, int m, int x, int n, int* out) {
  for (int i = 0; i < n; ++i) out[i] = steel::coord_item(units, nQB, range, m, x, i);
}
static steel::Problem problem(int S_q, int S_k, int D, int causal, int delta, int win) {
  steel::Problem p{};
  p.S_q = S_q; p.S_k = S_k; p.D = D; p.causal = causal; p.delta = delta; p.win_blocks = win;
  p.nQB = (S_q + 63) / 64; p.nKB = (S_k + 63) / 64;
  return p;
}
int range(int units, int nQB, int causal, int window, int single) {
  return steel::coord_range(units, problem(64 * nQB, 64 * nQB, 64, causal, 0, window), single);
}
int range_of(int units, int S_q, int S_k, int D, int causal) {
  return steel::coord_range(units, problem(S_q, S_k, D, causal, S_k - S_q, 0), 1);
}
int equal(int S_q, int S_k, int causal, int delta, int win) {
  return steel::equal_lists(problem(S_q, S_k, 64, causal, delta, win));
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    src, so = os.path.join(d, "order.hip"), os.path.join(d, "order.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-I", build.CSRC, src, "-o", so], check=True, capture_output=True)
    return ctypes.CDLL(so)


def share(lib, units, nQB, rng, x, m=1):
    n = lib.items(units, nQB, rng, x)
    out = (ctypes.c_int * (n + 1))()
    lib.order(units, nQB, rng, m, x, n + 1, out)
    assert out[n] == -1  # past the end
    return list(out[:n])


@pytest.mark.parametrize("nQB", [1, 2, 7, 8, 33, 130])
def test_every_item_once(lib, nQB):
    for units in list(range(1, 26)) + [36, 64, 100]:
        per = (units * nQB + 7) // 8  # positions the grids hold for an XCD
        for rng in [0] + [8 * r for r in range(1, (units + 7) // 8 + 1)]:
            for m in [m for m in (1, 2, 3, 5, 7) if units % m == 0]:
                shares = [share(lib, units, nQB, rng, x, m) for x in range(8)]
                assert all(len(s) <= per for s in shares)
                assert sorted(i for s in shares for i in s) == list(range(units * nQB)), (units, rng, m)


@pytest.mark.parametrize("units,nQB,causal,window,single", [
    (256, 32, False, False, True), (512, 32, True, False, True), (256, 64, True, True, True),
    (64, 32, False, False, False), (250, 32, False, False, True), (6, 512, True, True, True)])
def test_few_units_at_a_time(lib, units, nQB, causal, window, single):
    """What an XCD runs at one time (128 items) reads the keys and values of
    few units, where one range over all of them mixes up to units / 8 or more."""
    rng = lib.range(units, nQB, causal, window, single)
    most = 1 if rng == 0 else rng // 8
    assert most <= 16
    for x in range(8):
        s = [i // nQB for i in share(lib, units, nQB, rng, x)]
        # 128 items may straddle two ranges, and a last range that is no whole
        # eights is shared by all XCDs
        seen = max(len(set(s[i:i + 128])) for i in range(0, len(s), 64))
        assert seen <= (2 * most if rng == 0 or units % 8 == 0 else most + rng), (x, seen)


def test_small_calls_keep_one_range(lib):
    for units, nQB in ((1, 8), (96, 8), (8, 64), (16, 47), (24, 64)):
        assert lib.range(units, nQB, True, False, True) == (units + 7) // 8 * 8


@pytest.mark.parametrize("nQB", [8, 32, 47, 64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_ranges_are_of_about_one_size(lib, nQB, causal):
    """The last range, which begins with its heaviest lists when the others
    end, is no remainder of a unit or two per XCD."""
    for units in range(8, 600, 8):
        r = lib.range(units, nQB, causal, False, True) // 8
        last = units // 8 % r or r
        assert 2 * last >= r or r - last <= units // 8 // r, (units, r, last)


@pytest.mark.parametrize("groups", [8, 16, 64])
@pytest.mark.parametrize("m", [2, 3, 5, 7])
def test_units_of_a_group_share_an_xcd(lib, groups, m):
    """Heads that read the same keys and values run on one XCD."""
    units, nQB = groups * m, 16
    rng = lib.range(units, nQB, False, False, True)
    seen = {}
    for x in range(8):
        for i in share(lib, units, nQB, rng, x, m):
            seen.setdefault(i // nQB // m, set()).add(x)
    assert all(len(s) == 1 for s in seen.values())


@pytest.mark.parametrize("units,S_q,S_k,D", [(640, 256, 2816, 64), (384, 256, 15616, 64), (256, 256, 4096, 128),
                                             (512, 512, 2048, 128), (1280, 128, 3000, 64),
                                             (1024, 640, 1280, 128), (1024, 512, 768, 128)])
@pytest.mark.parametrize("causal", [False, True])
def test_query_blocks_of_a_unit_run_together(lib, units, S_q, S_k, D, causal):
    """Few query blocks against many keys: a unit's items lie within 1.5 ranges
    of 8 MiB of keys and values (or 8 units, 16 of unequal lists) of each other,
    so that they read them at one time."""
    nQB = -(-S_q // 64)
    least = 8 if lib.equal(S_q, S_k, causal, S_k - S_q, 0) else 16
    most = max(least, (8 << 20) // (S_k * D * 4))
    for x in range(8):
        s = [i // nQB for i in share(lib, units, nQB, lib.range_of(units, S_q, S_k, D, causal), x)]
        first, last = {}, {}
        for at, u in enumerate(s):
            first.setdefault(u, at)
            last[u] = at
        assert max(last[u] - first[u] for u in first) < 3 * most // 2 * nQB


@pytest.mark.parametrize("S_q,S_k,causal,delta,win", [
    (256, 2816, 1, 2560, 0), (512, 512, 1, 0, 0), (512, 2048, 1, 1536, 0), (1, 900, 1, 899, 0), (64, 900, 1, -30, 0),
    (512, 700, 0, 0, 0), (512, 512, 1, 0, 3), (300, 900, 1, 2000, 0), (300, 900, 1, -400, 0), (300, 900, 1, 100, 0),
    (100, 64, 1, -64, 0), (4096, 4096, 1, 0, 0), (1000, 12000, 1, 11000, 0), (1000, 12000, 1, -(1 << 30), 0),
    (1000, 12000, 1, 1 << 30, 0)])
def test_lists_of_about_one_length(lib, S_q, S_k, causal, delta, win):
    nQB, nKB = -(-S_q // 64), -(-S_k // 64)
    if causal and not win:
        lens = [min(nKB, max(0, -(-(min(64 * qb + 63, S_q - 1) + delta + 1) // 64))) for qb in range(nQB)]
        want = 4 * (max(lens) - min(lens)) <= max(lens)
    else:
        want = True
    assert bool(lib.equal(S_q, S_k, causal, delta, win)) == want
