"""The helper threads of large 3D reads (csrc/host_read.h): they touch the pages
of the result before there is data, without changing them, so that a read that
fails leaves the caller's arrays as they were; and they copy every chunk of
every plane, ragged last chunks and overlapping arrays included."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SOURCE = r"""
#include <chrono>
#include <cstdio>
#include "host_read.h"
using namespace lbk;

static int run(int planes, long long n, long long chunk, bool overlap) {
  HostRing ring;
  std::vector<double> slot[HostRing::SLOTS];
  for (int i = 0; i < HostRing::SLOTS; ++i) {
    slot[i].resize((size_t)planes * chunk);
    ring.mem[i] = (char *)slot[i].data();
  }
  std::vector<double> out((size_t)planes * n + 1), want;
  for (size_t i = 0; i < out.size(); ++i) out[i] = -(double)i - 1.0;
  std::vector<double *> h;
  for (int k = 0; k < planes; ++k) h.push_back(out.data() + (overlap ? 0 : (size_t)k * n));
  int bad = 0;
  want = out;
  {  // a read that fails before its first chunk
    HostCopiers c(ring, h.data(), planes, n, chunk);
    std::this_thread::sleep_for(std::chrono::milliseconds(30));
  }
  bad += out != want;
  {
    HostCopiers c(ring, h.data(), planes, n, chunk);
    const long long chunks = (n + chunk - 1) / chunk;
    for (long long j = 0; j < chunks; ++j) {
      c.wait(j - HostRing::SLOTS + 1);
      const long long n0 = j * chunk, cnt = std::min(chunk, n - n0);
      for (int k = 0; k < planes; ++k)
        for (long long i = 0; i < cnt; ++i) {
          const double v = 1000.0 * k + (double)(n0 + i);
          slot[j % HostRing::SLOTS][(size_t)k * cnt + i] = v;
          want[(overlap ? 0 : (size_t)k * n) + n0 + i] = v;
        }
      c.publish(j + 1);
    }
    c.wait(chunks);
  }
  bad += out != want;
  for (auto &m : ring.mem) m = nullptr;
  return bad;
}

int main() {
  int bad = 0;
  for (long long n : {1LL, 511LL, 512LL, 4096LL, 100003LL})
    for (int planes : {1, 4, 19})
      for (bool overlap : {false, true}) bad += run(planes, n, 1024, overlap);
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                    reason="no host compiler or HIP headers")
def test_helper_threads_leave_and_fill_the_arrays(tmp_path):
    src, exe = tmp_path / "read.cpp", tmp_path / "read"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "paper_2006_12910_amd", "csrc"),
                    str(src), "-o", str(exe), "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(ROCM, "lib")], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout.strip() == "0"
