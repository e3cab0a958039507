"""The joint launch of routing and gate/up on devices with fewer compute units (a partition of the GPU), on the CPU: a
program whose own definitions take the place of the runtime's occupancy queries asks the library."""
import os
import subprocess

from paper_2603_19289_amd import moe_spec as M

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2603_19289_amd")

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstdlib>
#include <dlfcn.h>
static int cus, per_cu;
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = cus; return hipSuccess; }
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = per_cu; return hipSuccess; }
int main(int argc, char **argv) {
  cus = std::atoi(argv[1]); per_cu = std::atoi(argv[2]);
  void *lib = dlopen(argv[3], RTLD_NOW | RTLD_GLOBAL);
  if (!lib) { std::puts(dlerror()); return 2; }
  auto supported = reinterpret_cast<bool (*)(int, int, int)>(dlsym(lib, "_ZN8moe_spec25route_gateup_b1_supportedEiii"));
  if (!supported) { std::puts(dlerror()); return 2; }
  for (int i = 4; i + 2 < argc; i += 3) std::printf("%d", supported(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2])));
  return 0;
}
"""


def test_joint_launch_is_taken_only_where_its_routing_workgroups_fit(tmp_path):
    src, exe = tmp_path / "ask.cpp", tmp_path / "ask"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", str(src), "-o", str(exe), "-ldl"], check=True)
    M.lib()                                                  # built, or the failure is about the build

    def ask(cus, per_cu, *shapes):
        args = [str(v) for shape in shapes for v in shape]
        done = subprocess.run([str(exe), str(cus), str(per_cu), os.path.join(PKG, "libmoe_spec.so")] + args, capture_output=True,
                              text=True, timeout=60, env=dict(os.environ, LD_LIBRARY_PATH=f"{rocm}/lib"))
        assert done.returncode == 0, done.stdout + done.stderr
        return done.stdout

    # (hidden, experts, dtype 1 = bf16): the whole device takes every number of experts, at the sizes the kernel is built for
    assert ask(256, 2, (2048, 256, 1), (4096, 256, 1), (4104, 8, 1), (2048, 256, 0), (2056, 8, 0)) == "11010"
    # 64 and 32 units: as many experts as two per workgroup that fits, and not one more
    assert ask(64, 2, (2048, 256, 1), (2048, 256, 0)) == "11"
    assert ask(64, 1, (2048, 128, 1), (2048, 129, 1), (1024, 127, 0), (2048, 192, 0)) == "1010"
    assert ask(32, 2, (2048, 128, 1), (512, 129, 1), (1024, 128, 0), (2048, 192, 0)) == "1010"
    assert ask(32, 3, (1024, 192, 0), (1024, 193, 0)) == "10"



ROUTING = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstdlib>
#include <dlfcn.h>
#include "kernels.h"
static int cus, per_cu, launched;
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = cus; return hipSuccess; }
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = per_cu; return hipSuccess; }
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
extern "C" hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { ++launched; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
int main(int argc, char **argv) {
  cus = std::atoi(argv[1]); per_cu = std::atoi(argv[2]);
  void *lib = dlopen(argv[3], RTLD_NOW | RTLD_GLOBAL);
  if (!lib) { std::puts(dlerror()); return 2; }
  auto launch = reinterpret_cast<hipError_t (*)(const moe_spec::RoutePairArgs &, int, hipStream_t)>(
      dlsym(lib, "_ZN8moe_spec17launch_route_pairERKNS_13RoutePairArgsEiP12ihipStream_t"));
  if (!launch) { std::puts(dlerror()); return 2; }
  for (int i = 4; i + 2 < argc; i += 3) {
    moe_spec::RoutePairArgs a{};
    a.B = std::atoi(argv[i]); a.E = std::atoi(argv[i + 1]); a.H = std::atoi(argv[i + 2]); a.k = 1;
    launched = 0;
    const hipError_t e = launch(a, 1, nullptr);
    std::printf("%c", e == hipErrorLaunchOutOfResources && !launched ? 'r' : e == hipSuccess && launched == 1 ? 'l' : '?');
  }
  return 0;
}
"""


def test_routing_that_does_not_fit_is_refused_before_it_is_launched(tmp_path):
    # what a short prompt relies on: it is then routed by the kernel for prompts, whose workgroups wait for nobody
    src, exe = tmp_path / "route.cpp", tmp_path / "route"
    src.write_text(ROUTING)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include", f"-I{PKG}/csrc", str(src), "-o", str(exe),
                    "-ldl"], check=True)
    M.lib()

    def ask(cus, per_cu, *shapes):
        args = [str(v) for shape in shapes for v in shape]
        done = subprocess.run([str(exe), str(cus), str(per_cu), os.path.join(PKG, "libmoe_spec.so")] + args, capture_output=True,
                              text=True, timeout=60, env=dict(os.environ, LD_LIBRARY_PATH=f"{rocm}/lib"))
        assert done.returncode == 0, done.stdout + done.stderr
        return done.stdout

    # (tokens, experts, hidden), bf16
    assert ask(256, 2, (1, 256, 2048), (64, 256, 2048), (1, 256, 4096)) == "lll"
    assert ask(32, 2, (1, 64, 2048), (1, 65, 2048), (64, 256, 2048), (2, 256, 2048), (1, 256, 1024)) == "lrllr"
