"""The pool of side streams, on the host against a stand-in of the runtime.

Every call that asks gets its stream however many others hold one and whatever
device they are on, idle ones are bounded per device, a runtime that has none
to give leaves no error behind, and a stream under capture is not forked from.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_06806_amd", "csrc")

RUNTIME = r"""
#pragma once
struct Obj { int device; };
typedef Obj* hipStream_t;
typedef Obj* hipEvent_t;
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2 };
inline int g_device, g_streams, g_events, g_limit = 1 << 30, g_record_fails;
inline bool g_capturing;
inline hipError_t g_last;
inline hipError_t ret(hipError_t e) { if (e != hipSuccess) g_last = e; return e; }
inline hipError_t hipGetLastError() { hipError_t e = g_last; g_last = hipSuccess; return e; }
inline hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  if (g_streams >= g_limit) return ret(hipErrorOutOfMemory);
  ++g_streams; *s = new Obj{g_device}; return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) { --g_streams; delete s; return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { ++g_events; *e = new Obj{g_device}; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { --g_events; delete e; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return ret(g_record_fails ? hipErrorUnknown : hipSuccess); }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess;
}
"""

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include <memory>
#include "side_stream.h"
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  Obj caller{0};
  {
    // four devices with eight calls' streams each, all held at once
    std::vector<std::unique_ptr<edx::SideStream>> held;
    for (g_device = 0; g_device < 4; ++g_device)
      for (int k = 0; k < 8; ++k) {
        held.push_back(std::make_unique<edx::SideStream>());
        CHECK(held.back()->fork(&caller));
        CHECK(held.back()->stream()->device == g_device);
      }
    for (size_t a = 0; a < held.size(); ++a)
      for (size_t b = 0; b < a; ++b) CHECK(held[a]->stream() != held[b]->stream());
    g_device = 0;
    for (int k = 0; k < 40; ++k) {
      held.push_back(std::make_unique<edx::SideStream>());
      CHECK(held.back()->fork(&caller));
    }
  }
  // idle ones: at most 16 a device, and events with them
  CHECK(g_streams == 16 + 3 * 8 && g_events == g_streams);
  {
    edx::SideStream again;
    CHECK(again.fork(&caller) && g_streams == 16 + 3 * 8);    // one that was kept
  }
  {
    // the same ones in the same order again, whatever order they came back in
    auto a = std::make_unique<edx::SideStream>(), b = std::make_unique<edx::SideStream>();
    CHECK(a->fork(&caller) && b->fork(&caller));
    hipStream_t first = a->stream(), second = b->stream();
    a.reset();
    b.reset();
    edx::SideStream c, d;
    CHECK(c.fork(&caller) && c.stream() == first && d.fork(&caller) && d.stream() == second);
  }
  // none to be had: the call goes on, and its next look at the last error is clean
  g_device = 5;
  g_limit = 0;
  {
    edx::SideStream s;
    CHECK(!s.fork(&caller) && hipGetLastError() == hipSuccess);
  }
  g_limit = 1 << 30;
  g_record_fails = 1;
  {
    edx::SideStream s;
    CHECK(!s.fork(&caller) && hipGetLastError() == hipSuccess);
  }
  g_record_fails = 0;
  g_capturing = true;
  {
    edx::SideStream s;
    CHECK(!s.fork(&caller));
  }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_side_streams(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = tmp_path / "main"
    r = subprocess.run(["g++", "-std=c++17", "-I", str(tmp_path), "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(exe),
                        "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_calls_take_their_streams_from_the_pool():
    """A stream made beside the kept ones may share the hardware queue of the
    caller's stream; only the server makes its own, for its lifetime."""
    made = [f for f in sorted(os.listdir(CSRC)) if "hipStreamCreate" in open(os.path.join(CSRC, f)).read()]
    assert made == ["serve.hip", "side_stream.h"]
