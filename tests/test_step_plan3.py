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
