"""How the steps of a call are split into launches (csrc/step_plan.h, host code):
the choice of region and steps a launch against measured times of every choice,
and the splits of every step count."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "step_plan.h"
using namespace lbk;
// the launches of a call of c steps: how many of each length, and the regions
extern "C" int plan(int st, int noise, int power, int plm, int nx, int ny, int c, int *len, int *k) {
  const MultiPlan p = plan_multi(StepKind{st, noise != 0, power != 0, plm}, Sizes{{nx, ny}});
  const StepSplit r = split_steps(c, p);
  for (int i = 0; i < r.parts; ++i) len[i] = r.len(i), k[i] = p.k[len[i]];
  return r.parts;
}
// with launches of up to nmax steps alone, of the same time a step each
extern "C" int split(int c, int nmax, int *len) {
  MultiPlan p;
  for (int n = 1; n <= nmax; n += 2) p.us[n] = n == nmax || n == 1 ? 1.0 : n == 3 ? 2.0 : 3.0;
  const StepSplit r = split_steps(c, p);
  for (int i = 0; i < r.parts; ++i) len[i] = r.len(i);
  return r.parts;
}
"""

# Measured on MI355X in sheared flow: us a launch of n steps over region k,
# {(k, n): us}; n = 1 (under region 1) the single-step sweep.
MEASURED = [
    ("f64 obst 128x64", {(0, 3): 4.9, (0, 5): 6.1, (0, 7): 6.9, (1, 1): 4.2, (1, 3): 7.1, (1, 5): 9.4, (1, 7): 11.4, (1, 9): 13.1}),
    ("f64 pl75 4096x4096", {(0, 3): 1520.5, (0, 5): 3789.6, (1, 1): 550.8, (1, 3): 1320.8, (1, 5): 2606.1}),
    ("f64 open 1448x1448", {(0, 3): 70.7, (0, 5): 100.3, (0, 7): 246.6, (1, 1): 57.1, (1, 3): 70.9, (1, 5): 90.3, (1, 7): 143.1, (1, 9): 243.4}),
    ("f64 noise 2048x2048", {(0, 3): 268.2, (0, 5): 620.8, (1, 1): 117.2, (1, 3): 250.4, (1, 5): 449.4}),
    ("f32 pl5 128x64", {(0, 3): 5.9, (0, 5): 7.7, (0, 7): 9.2, (1, 1): 4.8, (1, 3): 8.5, (1, 5): 11.9, (1, 7): 15.5, (1, 9): 18.4, (2, 3): 13.5, (2, 5): 19.3, (2, 7): 24.8, (2, 9): 29.3}),
    ("f32 open 4096x4096", {(0, 3): 349.7, (0, 5): 591.7, (1, 1): 226.4, (1, 3): 300.1, (1, 5): 446.5, (2, 3): 293.5, (2, 5): 419.1}),
    ("f32 obst 2048x2048", {(0, 3): 99.6, (0, 5): 175.7, (1, 1): 59.2, (1, 3): 86.2, (1, 5): 134.5, (2, 3): 89.3, (2, 5): 121.2}),
    ("f32 noise 512x512", {(0, 3): 12.9, (0, 5): 23.0, (0, 7): 51.5, (1, 1): 6.3, (1, 3): 13.6, (1, 5): 19.1, (1, 7): 31.5, (1, 9): 46.9, (2, 3): 15.1, (2, 5): 21.4, (2, 7): 39.9, (2, 9): 47.3}),
    ("f32 pl75 2048x2048", {(0, 3): 247.4, (0, 5): 574.4, (1, 1): 78.3, (1, 3): 219.9, (1, 5): 436.9, (2, 3): 230.7, (2, 5): 416.1}),
    ("f16 noise 2048x2048", {(0, 3): 141.8, (0, 5): 328.8, (1, 1): 38.4, (1, 3): 120.9, (1, 5): 242.5, (2, 3): 123.8, (2, 5): 227.2}),
    ("f16 obst 1448x1448", {(0, 3): 41.6, (0, 5): 88.5, (0, 7): 234.0, (1, 1): 19.0, (1, 3): 37.9, (1, 5): 68.7, (1, 7): 117.1, (1, 9): 205.4, (2, 3): 37.8, (2, 5): 61.9, (2, 7): 91.6, (2, 9): 149.5}),
    ("f16 pl75 4096x4096", {(0, 3): 986.2, (0, 5): 2425.1, (1, 1): 282.6, (1, 3): 861.4, (1, 5): 1755.4, (2, 3): 845.8, (2, 5): 1583.9}),
    ("bf16 obsnoise 2048x2048", {(0, 3): 148.7, (0, 5): 331.7, (1, 1): 44.9, (1, 3): 137.0, (1, 5): 272.5, (2, 3): 131.5, (2, 5): 222.9}),
    ("f16 pl5 4096x256", {(0, 3): 31.2, (0, 5): 67.4, (0, 7): 180.6, (1, 1): 13.1, (1, 3): 31.9, (1, 5): 57.0, (1, 7): 98.2, (1, 9): 166.7, (2, 3): 34.0, (2, 5): 61.8, (2, 7): 95.0, (2, 9): 133.3}),
    ("bf16 trt 724x700", {(0, 3): 12.1, (0, 5): 24.9, (0, 7): 60.7, (1, 1): 7.8, (1, 3): 12.8, (1, 5): 21.7, (1, 7): 36.4, (1, 9): 55.1, (2, 3): 16.1, (2, 5): 23.3, (2, 7): 29.7, (2, 9): 45.0}),
]


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2006_12910_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


def _launches(planner, name, c):
    storage, kind, size = name.split()
    nx, ny = (int(v) for v in size.split("x"))
    plm = {"pl13": 0, "pl5": 1, "pl75": 2}.get(kind, 0)
    lens, regions = (C.c_int * 4096)(), (C.c_int * 4096)()
    parts = planner.plan(["f64", "f32", "f16", "bf16"].index(storage), "noise" in kind, "pl" in kind, plm,
                         nx, ny, c, lens, regions)
    return lens[:parts], regions[:parts]


def _splits(c):
    """The splits that the plan chooses among: parts as few and as equal as a
    largest one allows, and five in place of one of three and two of one."""
    out = []
    for n in range(1, 10, 2):
        parts = -(-c // n)
        parts += (parts ^ c) & 1
        lo = c // parts
        lo -= 1 - lo % 2
        longer = (c - parts * lo) // 2
        lens = [lo + 2] * longer + [lo] * (parts - longer)
        out.append(lens)
        if n == 3 and lo == 1:
            f = min(longer, (parts - longer) // 2)
            out.append([5] * f + [3] * (longer - f) + [1] * (parts - longer - 2 * f))
    return out


@pytest.mark.parametrize("name,times", MEASURED)
def test_splits_are_near_the_best_measured_ones(planner, name, times):
    best_of = {n: min(t for (_, m), t in times.items() if m == n) for n in {m for _, m in times}}
    for c in (1, 2, 3, 4, 6, 8, 12, 16, 25, 50, 100, 250):
        lens, regions = _launches(planner, name, c)
        assert sum(lens) == c
        if any((k, n) not in times for n, k in zip(lens, regions) if n > 1):
            continue  # not measured: seven and nine steps on large lattices
        us = sum(times[(k, n) if n > 1 else (1, 1)] for n, k in zip(lens, regions))
        best = min(sum(best_of[n] for n in s) for s in _splits(c) if all(n in best_of for n in s))
        assert us <= 1.12 * best, (name, c, lens, us, best)


@pytest.mark.parametrize("nmax", [1, 3, 5, 7, 9])
def test_splits_are_odd_parts_that_add_up(planner, nmax):
    buf = (C.c_int * 4096)()
    for c in list(range(1, 200)) + [1023, 1024, 1025]:
        parts = planner.split(c, nmax, buf)
        lens = buf[:parts]
        assert sum(lens) == c and all(v % 2 == 1 and 1 <= v <= nmax for v in lens)
        assert lens == sorted(lens, reverse=True)
        assert parts <= -(-c // nmax) + 2
