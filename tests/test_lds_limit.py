"""CPU: a kernel's LDS limit is set once on every device that runs it.

csrc/lds_limit.h compiled against stand-ins for the two runtime calls."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

STUB = """
#pragma once
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
hipError_t hipGetDevice(int*);
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int);
"""
MAIN = """
#include "lds_limit.h"
#include <cstdio>
static int device, calls, fails;
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
  if (bytes != 90000) return hipErrorInvalidValue;
  ++calls;
  return fails-- > 0 ? hipErrorInvalidValue : hipSuccess;
}
static std::atomic<uint64_t> done{0};
static int use(int dev, int fail = 0) {  // runtime calls that one launch on dev makes; -1: it failed
  device = dev, calls = 0, fails = fail;
  return pd::allow_lds(nullptr, 90000, done) == hipSuccess ? calls : -1;
}
int main() {
  const int dev[] = {0, 0, 1, 1, 2, 2, 2, 63, 63, 64, 64};
  for (int k = 0; k < 11; ++k) std::printf("%d ", use(dev[k], k == 4));
}
"""


def test_every_device_once(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    subprocess.check_call(["g++", "-std=c++17", "-I" + str(tmp_path),
                           "-I" + os.path.join(ROOT, "paper_2604_12841_amd", "csrc"), str(tmp_path / "main.cpp"), "-o",
                           exe])
    # each device once, a failed call again, past 64 devices every time
    assert subprocess.check_output([exe], text=True).split() == "1 0 1 0 -1 1 0 1 0 1 1".split()
