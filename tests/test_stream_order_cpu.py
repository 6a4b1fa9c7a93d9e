"""The order of lbmrv_adjoint's work on its two streams, without a GPU.

A small C++ program drives the built library and answers its HIP calls itself:
a launch becomes an operation that happens after everything before it on its
stream, an event is what its stream had done when it was recorded, and a wait
adds that to another stream.  The header promises that the work on the
context's own stream is ordered against hip_stream by events in both
directions: it starts after what the caller queued before the call (which may
still be writing f0 or u~, or reading the same workspace) and is complete before
what is queued after it.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1312_3297_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <map>
#include <set>
#include <vector>
#include "lbmrv.h"

using Ops = std::set<int>;
struct Stream { Ops done; };
struct Event { Ops done; };
static Stream caller;                                // the caller's stream
static int next_op = 0;                              // never reused: a stale event names no later operation
static std::map<int, Ops> before;                    // operation -> what happens before it
static std::map<int, Stream*> on;                    // operation -> its stream
static Stream* of(hipStream_t s) { return reinterpret_cast<Stream*>(s); }

struct Config { dim3 grid, block; size_t shared; hipStream_t stream; };
static std::vector<Config> configs;

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
  configs.push_back({g, b, sh, s});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s) {
  const Config c = configs.back();
  configs.pop_back();
  *g = c.grid; *b = c.block; *sh = c.shared; *s = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) {
  before[next_op] = of(s)->done;
  on[next_op] = of(s);
  of(s)->done.insert(next_op++);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(new Stream); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete of(s); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new Event); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { reinterpret_cast<Event*>(e)->done = of(s)->done; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  const Ops& d = reinterpret_cast<Event*>(e)->done;
  of(s)->done.insert(d.begin(), d.end());
  return hipSuccess;
}
}

int main() {
  int fails = 0, second = 0;
  const double s9[9] = {0, 0, 0, 1.4, 1.7, 1.7, 1.2, 1.2, 1.4};
  std::vector<double> s19(19, 1.3);
  for (int k = 0; k <= 3; ++k) s19[k] = 0.0;
  char* p = reinterpret_cast<char*>(1 << 20);        // never dereferenced
  hipStream_t st = reinterpret_cast<hipStream_t>(&caller);
  // 2-D and 3-D; grids of one workgroup, of tiles and of pairs
  const struct { int lattice, storage; int64_t dims[3]; } grids[] = {
      {LBMRV_D2Q9, LBMRV_F32, {9, 9, 1}}, {LBMRV_D2Q9, LBMRV_F32, {70, 33, 1}}, {LBMRV_D2Q9, LBMRV_F64, {70, 33, 1}},
      {LBMRV_D3Q19, LBMRV_F32, {64, 64, 80}}, {LBMRV_D3Q19, LBMRV_F16DEV, {20, 20, 20}}};
  for (const auto& g : grids) {
    lbmrv_ctx* c = nullptr;
    const double* s = g.lattice == LBMRV_D2Q9 ? s9 : s19.data();
    if (lbmrv_create(&c, g.lattice, LBMRV_BASIS_DEFAULT, 1.0, s, g.dims, g.storage, 1.0) != LBMRV_OK) return 2;
    for (int64_t n = 1; n <= 26; ++n)
      for (int64_t K = 1; K <= n; ++K) {
        auto neighbour = [&] {  // any work of the caller's, one launch
          if (lbmrv_init_equilibrium(c, (double*)p, (double*)p, nullptr, 0.0, p, st) != LBMRV_OK) ++fails;
          return next_op - 1;
        };
        const int head = neighbour();
        if (lbmrv_adjoint(c, p, LBMRV_UT_FIELD, 1.0, (float*)p, n, K, p, p, (size_t)1 << 60, p, p, (double*)p, (double*)p, st) !=
            LBMRV_OK)
          ++fails;
        const int tail = neighbour();
        for (int o = head + 1; o < tail; ++o) {
          second += on[o] != &caller;
          if (!before[o].count(head)) {
            std::printf("lattice %d %lldx%lldx%lld steps %lld K %lld: launch %d does not wait for the caller's earlier work\n",
                        g.lattice, (long long)g.dims[0], (long long)g.dims[1], (long long)g.dims[2], (long long)n,
                        (long long)K, o - head);
            ++fails;
            break;
          }
        }
        for (int o = head + 1; o < tail; ++o)
          if (!before[tail].count(o)) {
            std::printf("lattice %d steps %lld K %lld: launch %d may outlast the call\n", g.lattice, (long long)n,
                        (long long)K, o - head);
            ++fails;
            break;
          }
        // the next call starts on a clean record
        const Stream* own = nullptr;
        for (int o = head + 1; o < tail; ++o)
          if (on[o] != &caller) own = on[o];
        if (own) const_cast<Stream*>(own)->done.clear();
        caller.done.clear();
        before.clear();
        on.clear();
      }
    lbmrv_destroy(c);
  }
  std::printf("%s (%d failed), %d launches on the second stream\n", fails ? "FAIL" : "OK", fails, second);
  return fails || !second;
}
"""


def test_adjoint_orders_its_second_stream_against_the_callers(tmp_path):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip")):
        pytest.skip("no C++ compiler or HIP headers")
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(DRIVER)
    # the program's own definitions of the HIP calls come before the runtime's
    cmd = ["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
           "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe), os.path.join(PKG, "liblbmrv.so"),
           "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[:3000] + r.stderr[-1000:]
    assert "OK (0 failed)" in r.stdout
