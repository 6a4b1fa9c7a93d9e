"""How lbmrv_step shares its steps among launches, without a GPU.

A small C++ program drives the built library and answers its HIP calls itself,
printing the kernel of every launch and, for k_tile, the steps it takes.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1312_3297_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
#include "lbmrv.h"

static std::map<const void*, std::string>& names() { static auto* m = new std::map<const void*, std::string>; return *m; }
struct Config { dim3 grid, block; size_t shared; hipStream_t stream; };
static std::vector<Config> configs;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
  names()[f] = name;
}
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
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  const std::string& n = names()[f];
  const size_t at = n.find("k_");
  unsigned steps = 0;
  if (n.compare(at, 6, "k_tile") == 0) std::memcpy(&steps, args[1], sizeof steps);  // first member of TileArgs
  std::printf(" %.6s:%u", n.c_str() + at, steps);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
}

// the monomials of the lattice's default basis as a run-time basis
static int create_run_time(lbmrv_ctx** c, int lattice, const double* s, const int64_t* dims, int storage) {
  static const int e[27][3] = {{0,0,0},{1,0,0},{0,1,0},{0,0,1},{2,0,0},{0,2,0},{0,0,2},{1,1,0},{0,1,1},{1,0,1},
                               {1,2,0},{1,0,2},{2,1,0},{0,1,2},{2,0,1},{0,2,1},{1,1,1},{2,2,0},{2,0,2},{0,2,2},
                               {2,1,1},{1,2,1},{1,1,2},{2,2,1},{2,1,2},{1,2,2},{2,2,2}};
  std::vector<int32_t> pot, ex;
  std::vector<double> co;
  for (const auto& m : e) {
    if (lattice == LBMRV_D2Q9 && m[2]) continue;
    if (lattice == LBMRV_D3Q19 && m[0] && m[1] && m[2]) continue;
    pot.push_back((int32_t)pot.size());
    ex.insert(ex.end(), m, m + 3);
    co.push_back(1.0);
  }
  const lbmrv_poly_basis pb{(int32_t)pot.size(), pot.data(), ex.data(), co.data()};
  return lbmrv_create_custom(c, lattice, &pb, 1.0, s, dims, storage, 1.0);
}

int main(int argc, char** argv) {
  // lattice storage nx ny nz most-steps run-time-basis
  const int lattice = std::atoi(argv[1]), storage = std::atoi(argv[2]);
  const int64_t dims[3] = {std::atoll(argv[3]), std::atoll(argv[4]), std::atoll(argv[5])};
  double s[27];
  for (int k = 0; k < 27; ++k) s[k] = k <= (lattice == LBMRV_D2Q9 ? 2 : 3) ? 0.0 : 1.3;
  lbmrv_ctx* c = nullptr;
  if ((std::atoi(argv[7]) ? create_run_time(&c, lattice, s, dims, storage)
                          : lbmrv_create(&c, lattice, LBMRV_BASIS_DEFAULT, 1.0, s, dims, storage, 1.0)) != LBMRV_OK)
    return 2;
  for (int64_t n = 1; n <= std::atoll(argv[6]); ++n) {
    std::printf("%lld:", (long long)n);
    if (lbmrv_step(c, (void*)(1 << 20), (void*)(1 << 24), LBMRV_UT_FLUID, 1.0, nullptr, n, nullptr) != LBMRV_OK) return 3;
    std::printf("\n");
  }
  lbmrv_destroy(c);
  return argc == 8 ? 0 : 4;
}
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip")):
        pytest.skip("no C++ compiler or HIP headers")
    d = tmp_path_factory.mktemp("launches")
    src, exe = d / "launches.cpp", d / "launches"
    src.write_text(DRIVER)
    # the program's own definitions of the HIP calls come before the runtime's
    cmd = ["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
           "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe), os.path.join(PKG, "liblbmrv.so"),
           "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(lattice, storage, shape, most, run_time=0):
        dims = (tuple(reversed(shape)) + (1,))[:3]
        r = subprocess.run([str(exe)] + [str(v) for v in (lattice, storage) + dims + (most, run_time)], capture_output=True,
                           text=True, timeout=60)
        assert r.returncode == 0, (r.returncode, r.stderr[-1000:])
        return {int(n): [(k, int(s)) for k, s in re.findall(r"(k_\w+):(\d+)", rest)]
                for n, rest in re.findall(r"^(\d+):(.*)$", r.stdout, re.M)}
    return run


# grids of tiles of 2, 3, 4 and 8 steps (D2Q9 = 0, D3Q19 = 1, D3Q27 = 2; f64 = 0, f32 = 1, f16dev = 3)
@pytest.mark.parametrize("lattice,storage,shape", [
    (2, 1, (15, 10, 15)), (2, 1, (27, 28, 31)), (2, 0, (10, 18, 15)), (1, 1, (41, 49, 44)), (1, 1, (10, 10, 10)),
    (1, 3, (24, 25, 26)), (0, 1, (64, 64)), (0, 0, (300, 301)), (0, 1, (2048, 2048))])
def test_few_tile_launches_take_one_step(launches, lattice, storage, shape):
    """A launch of k_tile for one step costs more than a single step and saves
    nothing.  At most two of them make the count of launches odd, and a call
    never has more launches than single steps need."""
    got = launches(lattice, storage, shape, 40)
    assert sorted(got) == list(range(1, 41))
    for n, seq in got.items():
        assert sum(s == 1 for k, s in seq if k == "k_tile") <= 2, (n, seq)
        assert len(seq) <= n + (n % 2 == 0), (n, seq)
        if n >= 2:
            assert any(k == "k_tile" for k, _ in seq), (n, seq)
            # every step is in one launch: k_tile's own, one in each other
            assert sum(s if k == "k_tile" else 1 for k, s in seq) == n, (n, seq)


# run-time bases: what each grid takes for 20 steps (the kernel that takes more than
# one step per launch, and the most steps of a launch), on both sides of each rule
@pytest.mark.parametrize("lattice,storage,shape,fused", [
    (1, 0, (16, 16, 16), ("k_tile", 3)), (1, 1, (20, 25, 27), ("k_tile", 3)), (1, 3, (24, 20, 20), ("k_tile", 3)),
    (1, 0, (32, 32, 32), ("k_tile", 2)), (1, 1, (32, 32, 32), ("k_tile", 2)), (1, 3, (20, 32, 32), ("k_tile", 2)),
    (1, 1, (48, 48, 48), None), (1, 0, (48, 48, 48), None), (1, 1, (64, 64, 64), None), (1, 3, (48, 48, 48), None),
    (1, 0, (96, 96, 96), None), (1, 1, (128, 128, 128), None),
    (2, 0, (16, 16, 16), ("k_tile", 2)), (2, 0, (20, 20, 20), None), (2, 1, (20, 20, 20), ("k_tile", 2)),
    (2, 1, (32, 32, 32), ("k_tile", 2)), (2, 3, (20, 20, 20), ("k_tile", 2)), (2, 0, (128, 128, 128), None),
    (2, 1, (96, 96, 96), None), (0, 1, (512, 512), ("k_tile", 5)), (0, 0, (64, 64), ("k_tile", 8))])
def test_run_time_bases_take_the_faster_kernel(launches, lattice, storage, shape, fused):
    """The dense relaxation makes ring nodes dear in space: D3Q27 FP32 96^3 took
    1925 us for 21 steps by pairs against 947 by single steps, D3Q19 FP32 64^3 296
    against 228 by tiles."""
    got = launches(lattice, storage, shape, 21, 1)
    for n in (20, 21):
        many = [(k, s) for k, s in got[n] if k == "k_slid" or s > 1]
        assert {k for k, _ in many} == ({fused[0]} if fused else set()), got[n]
        if fused:
            # 20 or 21 steps in an odd number of launches of at most that many each
            assert max(s for _, s in many) <= fused[1], got[n]
            assert len(got[n]) <= -(-n // fused[1]) + 1, got[n]
