"""CPU check of the rule that picks the class kernel's form (csrc/class_form.h) against measured times
of whole searches: [instances, layers, strategies, backpointers, tiles of the budget, tiles with work,
us with one launch per front, several fronts per launch with four waves per tile, with eight].  Random
shapes that the rule was not fitted to; MI355X."""
import ctypes
import json
import math
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "class_form.h"
extern "C" int warm(int B, int L, int SP, int bp, float used) {
  const gs::ClassForm f = gs::class_form(B, L, SP, bp != 0, used);
  return f.pays ? f.waves : 0;
}
extern "C" int cold(int B, int L, int SP, int bp, int tiles) {
  const gs::ClassForm f = gs::class_form_unknown(B, L, SP, bp != 0, tiles);
  return f.pays ? f.waves : 0;
}
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("class_form")
    (d / "form.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2504_21411_amd", "csrc"), str(d / "form.cpp"), "-o",
                    str(d / "form.so")], check=True)
    lib = ctypes.CDLL(str(d / "form.so"))
    lib.warm.argtypes = [ctypes.c_int] * 4 + [ctypes.c_float]
    return lib


def _times(name="class_form_times.json"):
    with open(os.path.join(ROOT, "tests", "data", name)) as f:
        return json.load(f)


def _padded(S):
    return next(v for v in (16, 24, 32, 48, 64, 96, 128, 192, 256) if S <= v)


def _ratios(pick, *name):
    out = []
    for B, L, S, bp, tiles, used, single, four, eight in _times(*name):
        t = {0: single, 4: four, 8: eight}[pick(B, L, _padded(S), bp, tiles, used)]
        out.append(t / min(single, four, eight))
    return out, math.exp(sum(map(math.log, out)) / len(out))


def test_the_form_picked_is_about_the_fastest(form):
    """With the tiles with work known (as an earlier solve's count and its margin)."""
    r, mean = _ratios(lambda B, L, SP, bp, tiles, used:
                      form.warm(B, L, SP, bp, float(min(tiles, used + max(4, used // 16)))))
    assert mean <= 1.015 and sum(x > 1.1 for x in r) <= 0.05 * len(r) and max(r) < 1.8, (mean, max(r))


def test_batches_beyond_the_fit(form):
    """158 to 2000 instances: on large loads one launch per front is the faster form, whatever the costs,
    which were fitted to smaller ones, would say.  (A first solve tries several fronts up to a tenth
    dearer.)"""
    warm = lambda B, L, SP, bp, tiles, used: form.warm(B, L, SP, bp, float(min(tiles, used + max(4, used // 16))))
    cold = lambda B, L, SP, bp, tiles, used: form.cold(B, L, SP, bp, tiles)
    for pick, most, share in ((warm, 1.015, 0.06), (cold, 1.03, 0.12)):
        r, mean = _ratios(pick, "class_form_times_large.json")
        assert mean <= most and sum(x > 1.1 for x in r) <= share * len(r) and max(r) < 1.4, (mean, max(r))
    assert form.warm(815, 27, 24, 1, 51.0) == 0 and form.cold(815, 27, 24, 1, 51) == 0


def test_the_first_solve_is_not_far_off(form):
    """Nothing known: the form tried costs little more, and only where it may turn out the faster."""
    r, mean = _ratios(lambda B, L, SP, bp, tiles, used: form.cold(B, L, SP, bp, tiles))
    assert mean <= 1.045 and max(r) < 2.2, (mean, max(r))


def test_a_form_without_four_waves_is_never_given_four(form):
    for SP in (192, 256):
        for bp in (0, 1):
            assert {form.warm(B, 24, SP, bp, float(t)) for B in (1, 8, 13, 64) for t in (1, 16, 120, 250)} <= {0, 8}
