"""Host side of the resident launches (resident_host.cpp) on the CPU: built
with the host compiler against the HIP headers and run with stand-ins for the
calls it makes and for the kernels."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"

STAND_INS = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "resident_host.hpp"
using namespace femheat;

static int limit_set = 64 * 1024;  // dynamic LDS that the one kernel may be launched with
static void (*between)() = nullptr;  // what another thread does between the limit and the launch
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int value) {
  limit_set = value;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t lds, hipStream_t) {
  if (between) {
    auto f = between;
    between = nullptr;
    f();
  }
  return lds <= (size_t)limit_set ? hipSuccess : hipErrorInvalidValue;
}
namespace femheat {
const void* resident_kernel_f64(int, int) { return "f64"; }
const void* resident_kernel_mixed(int, int) { return "mixed"; }
const void* resident_kernel_cheb(int, int) { return "cheb"; }
}
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s\n", #x); return 1; } } while (0)
"""


def run(tmp_path, body):
    if not os.path.exists(CLANG):
        pytest.skip("LLVM clang++ not found")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(STAND_INS + body)
    csrc = os.path.join(ROOT, "paper_1905_07622_amd", "csrc")
    cmd = [CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
           os.path.join(ROOT, "include"), "-I", csrc, str(src), os.path.join(csrc, "resident_host.cpp"), "-o", str(exe),
           "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_another_threads_launch_does_not_lower_the_lds_limit(tmp_path):
    """A launch of the same kernel with less LDS, made by another thread
    between this launch's limit and the launch itself."""
    run(tmp_path, r"""
static hipError_t launch(size_t lds) { return resident_launch(RES_F64, 0, 9, 8, 512, lds, nullptr, nullptr, nullptr); }
int main() {
  between = [] { if (launch(16 * 1024) != hipSuccess) std::abort(); };
  CHECK(launch(kResLds) == hipSuccess);
  return 0;
}
""")


@pytest.mark.parametrize("n", [1, 2, 64, 1023, 1024, 1025, 65535, 65536, 1000000])
def test_reset_grid_fits_any_number_of_simulations(tmp_path, n):
    run(tmp_path, f"""
int main() {{
  for (uint32_t nodes : {{8u, 257u, 1u << 20}}) {{
    const dim3 g = resident_reset_grid({n}u, nodes);
    CHECK(g.x >= 1 && g.y >= 1 && g.z == 1 && g.y <= 65535u && (uint64_t)g.x * g.y <= 16384);
    CHECK({n}u > 65535u || g.y == std::min({n}u, 1024u));
  }}
  return 0;
}}
""")
