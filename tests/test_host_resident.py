"""Admission of the one-launch coarse solves (csrc/resident.h), built with the host compiler: a
launch waits for room within its bound and is turned away after it."""
import os
import shutil
import subprocess

import pytest

from _support import ROOT

MAIN = r"""
#include <cstdio>
#include <thread>

#include "resident.h"
using hpmg::ResidentGroups;
using Clock = std::chrono::steady_clock;

static double since(Clock::time_point t) { return std::chrono::duration<double>(Clock::now() - t).count(); }
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

int main() {
  {
    ResidentGroups a(0, 200, 256, 0.0);
    CHECK(a.admitted());
    const auto t = Clock::now();
    ResidentGroups b(0, 100, 256, 0.05);  // a never leaves meanwhile
    CHECK(!b.admitted() && since(t) >= 0.05 && since(t) < 5.0);
    ResidentGroups c(0, 56, 256, 0.0), other(1, 256, 256, 0.0);  // b holds nothing; devices are apart
    CHECK(c.admitted() && other.admitted());
    CHECK(!ResidentGroups(0, 1, 256, 0.0).admitted());
  }
  ResidentGroups all(0, 256, 256, 0.0);  // everything was given back
  CHECK(all.admitted());
  CHECK(!ResidentGroups(64, 1, 256, 0.0).admitted() && !ResidentGroups(-1, 1, 256, 0.0).admitted());
  {
    // room that comes within the bound is taken
    auto *held = new ResidentGroups(2, 200, 256, 0.0);
    bool in = false;
    std::thread waiter([&] { in = ResidentGroups(2, 100, 256, 60.0).admitted(); });
    std::this_thread::sleep_for(std::chrono::milliseconds(20));
    delete held;
    waiter.join();
    CHECK(in);
  }
  std::puts("ok");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_admission(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    csrc = os.path.join(ROOT, "paper_2204_01722_amd", "csrc")
    res = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-pthread", "-I", csrc, str(src), "-o",
                          str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
