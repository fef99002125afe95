"""How the 3D sweeps are run (csrc/step_plan3.h, host code), against measured
times of the choices."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "step_plan3.h"
using namespace lbk3;
extern "C" int two_steps(int st, int q, int solids, int trt, int power, double n, int nx, int ny, int nz) {
  return two_steps_pay3(Kind3{st, q, solids != 0, trt != 0, power != 0, n}, nx, ny, nz);
}
extern "C" int split(int st, int nx, int ny, int nz, int *planes) {
  const X2Split r = split3(st, nx, ny, nz);
  *planes = r.planes;
  return r.tiles;
}
extern "C" int streams(int q, int nx, int ny, int nz, int elem) { return streams3(q, nx, ny, nz, elem); }
"""
ELEM = {"f64": 8, "f32": 4, "f16": 2}

# us a step: single steps that keep to the last-level cache / stream past it
STREAM = [
    ("f64 d3q19 8x8x4096", 38.4, 55.6), ("f64 d3q27 8x8x4096", 53.2, 80.1),
    ("f32 d3q27 8x8x4096", 31.8, 46.3), ("f64 d3q27 16x256x64", 27.8, 38.6),
    ("f32 d3q19 250x99x33", 21.4, 29.1), ("f16 d3q27 64x64x512", 37.5, 49.7),
    ("f16 d3q19 192x192x130", 79.1, 69.2), ("f16 d3q19 65x401x101", 90.9, 66.2),
    ("f32 d3q19 192x192x130", 149.5, 136.0), ("f32 d3q19 65x401x101", 152.1, 121.4),
    ("f16 d3q27 192x192x130", 111.5, 98.0), ("f64 d3q19 130x130x130", 178.3, 145.9),
]

# us a step: single steps / two steps a launch, sheared flow (pl5, pl75, pl13:
# power law of n = 0.5, 0.75, 1.3; s: solids; t: TRT)
TWO = [
    ("f32 d3q19 open 192x192x130", 136.0, 99.3), ("f32 d3q19 pl75s 192x192x130", 150.8, 165.6),
    ("f32 d3q19 pl75 250x99x33", 22.4, 27.5), ("f32 d3q19 pl5s 400x30x100", 32.4, 36.6),
    ("f32 d3q19 pl5ts 250x99x33", 25.4, 27.6), ("f32 d3q27 pl5s 160x160x96", 113.3, 136.9),
    ("f32 d3q27 pl75s 256x160x128", 253.0, 275.8), ("f32 d3q27 pl13s 64x64x512", 94.3, 104.7),
    ("f32 d3q27 open 250x99x33", 29.7, 24.1), ("f32 d3q19 s 256x160x128", 171.8, 117.3),
    ("f64 d3q27 ts 64x64x64", 19.6, 21.1), ("f64 d3q19 open 128x128x32", 25.4, 19.9),
    ("f64 d3q27 s 192x192x130", 410.4, 270.1), ("f32 d3q19 open 33x33x17", 3.6, 8.0),
    ("f64 d3q19 open 8x8x4096", 38.4, 52.6), ("f32 d3q19 t 65x401x101", 121.5, 91.7),
]


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan3")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2006_12910_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


def _sizes(name):
    storage, lattice, size = name.split()[0], name.split()[1], name.split()[-1]
    return storage, int(lattice[3:]), tuple(int(v) for v in size.split("x"))


@pytest.mark.parametrize("name,cached,streaming", STREAM)
def test_streaming_where_it_is_the_faster(planner, name, cached, streaming):
    storage, q, size = _sizes(name)
    chosen = streaming if planner.streams(q, *size, ELEM[storage]) else cached
    assert chosen == min(cached, streaming)


@pytest.mark.parametrize("name,single,two", TWO)
def test_two_steps_a_launch_where_they_are_the_faster(planner, name, single, two):
    storage, q, size = _sizes(name)
    kind = name.split()[2]
    n = {"pl5": 0.5, "pl75": 0.75, "pl13": 1.3}.get(kind.rstrip("ts"), 1.0)
    planner.two_steps.argtypes = [C.c_int] * 5 + [C.c_double] + [C.c_int] * 3
    flags = "" if kind == "open" else kind.replace("pl", "")
    takes = planner.two_steps(["f64", "f32"].index(storage), q, "s" in flags, "t" in flags,
                              kind.startswith("pl"), n, *size)
    assert (two if takes else single) <= 1.03 * min(single, two)


@pytest.mark.parametrize("storage", [0, 1])
def test_segments_cover_the_walk(planner, storage):
    planes = C.c_int()
    for nz in list(range(1, 140)) + [4096]:
        tiles = planner.split(storage, 200, 101, nz, C.byref(planes))
        assert tiles == 4 * 21 and 1 <= planes.value <= nz
        segs = -(-nz // planes.value)
        assert (segs - 1) * planes.value < nz  # no empty segment
        assert segs == 1 or planes.value >= 4
