"""The host's wait for words that kernels store in pinned memory (wait_pinned), on the CPU against
a counting stand-in for the stream: how often it asks the stream, and that it ends by itself when
the stream's work ends or fails without the word."""
import os
import subprocess

import pytest

from tests.conftest import ROOT

SOURCE = r"""
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include "rpb_internal.h"

using Clock = std::chrono::steady_clock;
static long asked = 0;
static hipError_t answer = hipErrorNotReady;
extern "C" hipError_t hipStreamQuery(hipStream_t) { ++asked; return answer; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" const char *hipGetErrorString(hipError_t) { return "stand-in"; }
namespace rpb {
int fail(rpb_ctx *, int status, const char *, ...) { return status; }
}

int main() {
  const auto t0 = Clock::now();
  auto ms = [&] { return std::chrono::duration<double, std::milli>(Clock::now() - t0).count(); };
  // the word is there: no question to the stream
  int st = rpb::wait_pinned(nullptr, nullptr, [] { return true; });
  std::printf("%d %ld\n", st, asked);
  // the word arrives after a while
  const double until = ms() + 20.0;
  st = rpb::wait_pinned(nullptr, nullptr, [&] { return ms() >= until; });
  std::printf("%d %ld\n", st, asked);
  // the work ends without it, and fails
  answer = hipSuccess;
  std::printf("%d\n", rpb::wait_pinned(nullptr, nullptr, [] { return false; }));
  answer = hipErrorUnknown;
  std::printf("%d\n", rpb::wait_pinned(nullptr, nullptr, [] { return false; }));
  // the work ends and the word came with it
  answer = hipSuccess;
  const long before = asked;
  std::printf("%d\n", rpb::wait_pinned(nullptr, nullptr, [&] { return asked > before; }));
  return 0;
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("wait")
    src, exe = d / "wait.cpp", d / "wait"
    src.write_text(SOURCE)
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_1612_00474_amd", "csrc"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")]
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w",
                    *[f"-I{p}" for p in inc], str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60)
    return [[int(x) for x in line.split()] for line in r.stdout.splitlines()]


def test_the_stream_is_asked_seldom(lines):
    assert lines[0] == [0, 0]
    st, asked = lines[1]
    # 20 ms: a question per millisecond, where one every few microseconds slows the stream down
    assert st == 0 and asked <= 25, asked


def test_the_wait_ends_without_the_word(lines):
    assert lines[2] == [-3] and lines[3] == [-3]   # RPB_EDEVICE
    assert lines[4] == [0]
