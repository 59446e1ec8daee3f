"""How long the parts of the weight gradients' sums are (csrc/wgrad_plan.h, built with g++; the cut that every workgroup derives from the plan and
the selection is restated here).  A launch waits for its longest part, so no selection may leave one longer than cutting the token axis
of each of an expert's (sample, slot) pairs into the same number of ranges would, or cutting the list of pairs where there are many."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_02495_amd", "csrc")
SHIM = """
#include "wgrad_plan.h"
static void give(const uoe::WgradPlan &w, int *o) { o[0] = w.chunks; o[1] = w.items; o[2] = w.parts; o[3] = w.lo; o[4] = w.hi; o[5] = w.each; }
extern "C" void any_plan(int b, int l, int d, int n, int k, int s, int f32, int *o) { give(uoe::uome_any_wgrad(b, l, d, n, k, s, f32 != 0), o); o[6] = uoe::uome_any_range(l, o[1]); }
extern "C" void grid_plan(int b, int l, int d, int n, int k, int d_e, int *o) { give(uoe::uome_backward_wgrad(b, l, d, n, k, d_e), o); o[6] = l / o[1]; }
extern "C" void patch_plan(int b, int n, int k, int c, int l_p, int sets, int rows, int cols, int *o) { give(uoe::smha_backward_wgrad(b, n, k, c, l_p, sets, rows, cols), o); }
extern "C" void any_patch_plan(int b, int n, int k, int c, int l_p, int s, int *o) { give(uoe::smha_any_wgrad(b, n, k, c, l_p, s, 1024), o); }
"""


def build(d):
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cc"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return build(tmp_path_factory.mktemp("plan"))


def call(fn, *args):
    out = (ctypes.c_int * 7)()
    fn(*args, out)
    return dict(zip(("chunks", "items", "parts", "lo", "hi", "each", "range"), out))


def selections(rng, b, n, k):
    """Pairs an expert: even, random, and skewed to the first experts."""
    yield np.bincount(np.arange(b * k) % n, minlength=n)
    for weight in (np.ones(n), 1.0 / np.arange(1, n + 1)):
        yield np.bincount(np.concatenate([rng.choice(n, k, replace=False, p=weight / weight.sum()) for _ in range(b)]), minlength=n)


def longest(plan, lengths, counts, lookup=0):
    """Tokens of the longest part, `lookup` more for each item; lengths: tokens of a pair's items, counts: pairs an expert."""
    items = counts * plan["items"]
    if plan["each"]:
        per = -(-items // plan["each"])
        cuts = [np.minimum(np.arange(plan["each"] + 1) * p, i) for i, p in zip(items, per)]
    else:
        step = (plan["hi"] - plan["lo"] + 62) // 63
        tried = [min(plan["lo"] + lane * step, plan["hi"]) for lane in range(64)]
        fits = [p for p in tried if sum(-(-items // p)) <= plan["parts"]]
        assert fits
        parts = -(-items // fits[0])
        cuts = [np.arange(p + 1) * i // max(p, 1) for i, p in zip(items, parts)]
    most = 0
    for c, cut in zip(counts, cuts):
        ends = np.concatenate([[0], np.cumsum(np.tile(lengths + lookup, c))])
        assert cut[-1] == c * plan["items"] and np.diff(cut).max(initial=0) <= 128
        most = max(most, int(np.diff(ends[cut]).max(initial=0)))
    return most


ANY = [(8, 512, 8, 4, 8), (4, 770, 5, 2, 8), (6, 1000, 6, 3, 7), (10, 500, 5, 2, 8), (128, 196, 6, 3, 7), (24, 500, 4, 2, 6), (3, 2009, 13, 3, 4), (2, 64, 4, 2, 8),
       (1, 4096, 32, 1, 8), (16, 140, 12, 5, 3), (57, 128, 11, 4, 2), (100, 77, 4, 2, 5), (128, 300, 32, 7, 8), (12, 2500, 4, 1, 8), (5, 31, 3, 2, 4)]


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("b,l,n,k,s", ANY)
def test_any_shape(shim, b, l, n, k, s, f32):
    """K-steps are 32 tokens, a segment's lookups cost as much as 16 (4 in fp32)."""
    plan, lookup = call(shim.any_plan, b, l, 8, n, k, s, f32), 4 if f32 else 16
    assert plan["parts"] == n * s
    lengths = np.minimum(plan["range"], l - np.arange(plan["items"]) * plan["range"])
    assert lengths.min() > 0 and lengths.sum() == l and (plan["items"] == 1 or plan["range"] % 32 == 0)
    up = lambda v: -(-v // 32) * 32
    axis = min(up(l), up(-(-l // s)))
    got, want = [], []
    rng = np.random.default_rng(l)
    for _ in range(60):
        for counts in selections(rng, min(b, 128), n, k):
            got.append(longest(plan, up(lengths), counts, lookup))
            want.append(-(-counts.max() // s) * (up(l) + lookup) if b * k >= 4 * n * s else counts.max() * (axis + lookup))
    assert np.mean(got) <= 1.03 * np.mean(want), plan
    if f32 and plan["each"] and (b, l) in ((8, 512), (6, 1000)):
        assert all(np.asarray(got) <= np.asarray(want)), plan


@pytest.mark.parametrize("b,l,n,k,s", [(3, 4400, 4, 2, 8), (2, 30000, 5, 2, 8), (9, 1364, 16, 5, 4), (16, 1504, 16, 6, 4), (12, 2500, 4, 1, 8)])
def test_equal_parts_are_used(shim, b, l, n, k, s):
    """Parts that stay empty make the others, and the fp32 sums along them, longer."""
    plan = call(shim.any_plan, b, l, 8, n, k, s, 0)
    rng = np.random.default_rng(l)
    for _ in range(20):
        for counts in selections(rng, b, n, k):
            assert longest(plan, np.full(plan["items"], plan["range"]), counts) <= 1.6 * b * k * l / (n * s), (plan, counts)


GRID = [(8, 512, 512, 8, 4, 256), (8, 512, 512, 8, 3, 256), (4, 8192, 1024, 16, 8, 256), (16, 4096, 256, 8, 2, 128), (64, 512, 256, 4, 2, 128), (57, 128, 96, 11, 4, 64),
        (6, 2048, 32, 6, 2, 64), (24, 512, 32, 4, 2, 32), (4, 640, 128, 8, 1, 96), (3, 2720, 416, 12, 5, 96), (128, 1024, 64, 6, 3, 64), (32, 960, 160, 14, 2, 32)]


@pytest.mark.parametrize("b,l,d,n,k,d_e", GRID)
def test_on_the_32_grid(shim, b, l, d, n, k, d_e):
    plan = call(shim.grid_plan, b, l, d, n, k, d_e)
    s, axis = plan["parts"] // n, 1
    assert plan["range"] * plan["items"] == l and (plan["items"] == 1 or plan["range"] % 64 == 0)
    while 2 * axis <= s and l % (2 * axis * 64) == 0:
        axis *= 2
    rng = np.random.default_rng(l)
    for _ in range(20):
        for counts in selections(rng, b, n, k):
            assert longest(plan, np.full(plan["items"], plan["range"]), counts) <= counts.max() * (l // axis), (plan, counts)


@pytest.mark.parametrize("b,l,n,k,c,m,width,d,sets,own", [(14, 2688, 12, 5, 19, 84, 128, 160, 4, True), (6, 4096, 8, 4, 32, 128, 128, 256, 4, True), (9, 3072, 5, 3, 20, 96, 128, 384, 4, True),
                                                           (4, 4096, 3, 2, 32, 64, 128, 640, 4, True), (10, 1568, 11, 5, 16, 49, 32, 64, 4, False), (14, 2688, 12, 5, 19, 84, 96, 160, 2, False)])
def test_picked_patches_fill_the_last_round(shim, b, l, n, k, c, m, width, d, sets, own):
    """128 x 128 tiles on 256 compute units: a second round for a few tiles takes as long as a full one, unless d_x's tiles share the launch."""
    plan = call(shim.patch_plan, b, n, k, c, l // m, sets, width, d)
    an_expert = sets * n * -(-width // 128) * -(-d // 128)
    tiles = an_expert * plan["parts"] // n
    if own:
        assert tiles <= 128 or tiles % 256 == 0 or tiles % 256 >= 192 or plan["parts"] >= n * min(8, b * k * c // n // 8)
    else:
        assert 256 <= tiles < 256 + an_expert, plan


@pytest.mark.parametrize("b,n,k,c,l_p,s,equal", [(57, 12, 1, 7, 35, 3, True), (10, 13, 4, 6, 43, 2, True), (9, 5, 2, 7, 37, 3, True), (33, 9, 1, 5, 42, 2, True), (8, 8, 4, 4, 32, 2, False),
                                                       (4, 4, 2, 3, 15, 3, False), (128, 6, 3, 4, 14, 8, False)])
def test_any_shape_patches_in_equal_parts(shim, b, n, k, c, l_p, s, equal):
    """Where an unequal selection makes the longest part 128 tokens and more longer than an equal one; few tokens, or many pairs an expert, are not worth finding them."""
    assert (call(shim.any_patch_plan, b, n, k, c, l_p, s)["each"] == 0) == equal


def test_parts_fit_the_groups_coding(shim):
    """At most 8192 parts a chunk (13 bits), 256 where they are placed by sample: all sizes that the entry points accept (n * m <= 8192, n <= 32, b * m and b * k <= 65535)."""
    rng, most = np.random.default_rng(3), 0
    for _ in range(20000):
        n = int(rng.integers(1, 33))
        m = min(8192 // n, 1024)
        c, b = (m, min(65535 // m, 128)) if rng.random() < 0.3 else (int(rng.integers(1, m + 1)), int(rng.integers(1, 129)))
        k, d, w, l = int(rng.integers(1, n + 1)), 8 * int(rng.integers(1, 200)), 8 * int(rng.integers(1, 33)), int(2 ** rng.uniform(5, 16))
        parts = call(shim.patch_plan, b, n, k, c, 32, int(rng.choice([2, 4])), w, d)["parts"]
        most = max(most, parts)
        assert parts <= 8192, (b, n, k, c)
        plan = call(shim.grid_plan, b, l // 32 * 32, d, n, k, w)
        any_plan = call(shim.any_plan, b, l, d, n, k, int(rng.integers(1, 9)), int(rng.integers(0, 2)))
        assert plan["parts"] <= 256 and any_plan["parts"] <= 256, (b, l, d, n, k, w)
        assert (min(b, 128) - 1) * any_plan["items"] < 1 << 24 and any_plan["items"] <= 1024   # keys and contexts
    assert most >= 4096
