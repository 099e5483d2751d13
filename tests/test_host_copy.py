"""Device-to-host copies of whole fields, on the CPU: host_copy.cpp is built
against a stand-in for the runtime whose streams run their work late and in
order, and whose per-thread stream is another one in every thread, as HIP's
is."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_04606_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <stddef.h>
#include <stdlib.h>
#include <string.h>
#include <deque>
#include <functional>
#include <map>
#include <mutex>
#include <thread>
typedef int hipError_t;
typedef struct ihipStream_t *hipStream_t;
typedef struct Event *hipEvent_t;
enum { hipSuccess = 0, hipErrorOther = 1, hipHostMallocDefault = 0, hipEventDisableTiming = 2, hipMemcpyDeviceToHost = 2 };
#define hipStreamPerThread ((hipStream_t)2)
typedef std::pair<hipStream_t, std::thread::id> Queue;
struct Event { Queue q; };
inline std::recursive_mutex mu;
inline std::map<Queue, std::deque<std::function<void()>>> work;
inline Queue queue_of(hipStream_t s) { return {s, s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()}; }
inline void push(hipStream_t s, std::function<void()> f) { std::lock_guard<std::recursive_mutex> l(mu); work[queue_of(s)].push_back(f); }
inline void drain(Queue q) {
  std::lock_guard<std::recursive_mutex> l(mu);
  for (auto &w = work[q]; !w.empty(); w.pop_front()) w.front()();
}
inline hipError_t hipHostMalloc(void **p, size_t n, int) { *p = malloc(n); return *p ? 0 : 1; }
inline hipError_t hipHostFree(void *p) { free(p); return 0; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, int) { *e = new Event(); return 0; }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return 0; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { e->q = queue_of(s); return 0; }
inline hipError_t hipEventSynchronize(hipEvent_t e) { drain(e->q); return 0; }
inline hipError_t hipGetLastError() { return 0; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
inline hipError_t hipSetDevice(int) { return 0; }
inline hipError_t hipStreamSynchronize(hipStream_t s) { drain(queue_of(s)); return 0; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t st) { push(st, [=] { memcpy(d, s, n); }); return 0; }
"""

PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "host_copy.h"
// A kernel fills the device arrays on the caller's stream, then they are copied out.
int main(int argc, char **argv) {
  hipStream_t s = (hipStream_t)strtoul(argv[1], nullptr, 0);
  const size_t sizes[3] = {strtoul(argv[2], nullptr, 0), 1, 12345};
  const size_t gap = strtoul(argv[3], nullptr, 0);  // between the pieces on the device
  sbt::HostCopy copy;
  for (int pass = 0; pass < 2; ++pass) {
    std::vector<char> dev(sizes[0] + sizes[1] + sizes[2] + 2 * gap);
    std::vector<std::vector<char>> host, want;
    sbt::HostCopy::Piece pc[3];
    size_t at = 0;
    for (size_t n : sizes) host.emplace_back(n, 1), want.emplace_back(n, 1);
    for (int i = 0; i < 3; at += sizes[i++] + gap) {
      pc[i] = {dev.data() + at, host[i].data(), sizes[i]};
      for (size_t k = 0; k < sizes[i]; ++k) want[i][k] = (char)((at + k) * 31 + 7 + pass);
    }
    push(s, [&] { for (size_t i = 0; i < dev.size(); ++i) dev[i] = (char)(i * 31 + 7 + pass); });
    if (copy.to_host(pc, 3, s) != hipSuccess) return 2;
    if (host != want) { puts("copied before the kernel"); return 1; }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_copy")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(PROGRAM)
    exe = str(d / "copy")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-I", str(d), "-I", CSRC, str(d / "main.cpp"),
                    os.path.join(CSRC, "host_copy.cpp"), "-lpthread", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("gap", [0, 8])
@pytest.mark.parametrize("nbytes", [1000, (4 << 20) + 5, 11 << 20])
@pytest.mark.parametrize("stream", ["0", "2", "0x1000"], ids=["default", "per_thread", "own"])
def test_copies_follow_the_callers_stream(program, stream, nbytes, gap):
    """The default stream, the per-thread stream and one of the program's own,
    below and above the size from which several threads copy, pieces that lie
    together on the device and apart."""
    r = subprocess.run([program, stream, str(nbytes), str(gap)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
