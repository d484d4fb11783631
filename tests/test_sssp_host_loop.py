"""The host side of the SSSP search against a stand-in for the GPU, on the CPU:
its host code is linked with a small runtime whose stream runs the launched
steps one by one on a clock of its own.  The time limit counts from the search's
first step, whatever the stream had to do before it, and the mapped buffer that
queued steps write is not given back before they have run."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1506_03265_amd as cd

CSRC = os.path.join(os.path.dirname(os.path.abspath(cd.__file__)), "csrc")

RUNTIME = r"""
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <string>
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include "cldiam.h"

static double elapsed = 0;             // the clock, in seconds
static double begins = 0, ends = 0;    // the first step runs at `begins`, the search is done at `ends`
static std::map<const void *, std::string> names;
static std::deque<uint32_t> queued;    // steps on the stream
static volatile uint32_t mirror[1024];
static int fail_max = 0;               // k_sssp_max does not launch
static hipError_t error = hipSuccess;

static void run_step() {
  mirror[0] = queued.front();
  if (elapsed >= ends) mirror[1] = 1;
  queued.pop_front();
}
static void tick() {
  elapsed += 0.01;
  if (elapsed >= begins && !queued.empty()) run_step();
}
namespace std { namespace chrono { inline namespace _V2 {
steady_clock::time_point steady_clock::now() noexcept {
  tick();
  return time_point(nanoseconds((long long)(elapsed * 1e9)));
}
}}}
extern "C" int sched_yield() { tick(); return 0; }

extern "C" {
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *name, const char *, unsigned, void *, void *, void *, void *, int *) {
  names[f] = name;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
  const std::string &name = names[f];
  if (name.find("k_sssp_step") != std::string::npos) queued.push_back(*(uint32_t *)args[1]);
  if (fail_max && name.find("k_sssp_max") != std::string::npos) error = hipErrorLaunchFailure;
  return error;
}
hipError_t hipGetLastError() { const hipError_t e = error; error = hipSuccess; return e; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  if (elapsed < begins) elapsed = begins;
  while (!queued.empty()) { elapsed += 0.01; run_step(); }
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *, size_t n, hipMemcpyKind, hipStream_t) {
  hipStreamSynchronize(nullptr);
  memset(to, 0, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
}
namespace cld {
void set_error(const char *, ...) {}
int hip_fail(hipError_t, const char *) { return CLDIAM_EHIP; }
void *pinned_acquire(size_t) { return (void *)mirror; }
void pinned_release(void *) { printf("released with %zu steps queued\n", queued.size()); }
}

int main(int argc, char **argv) {
  begins = atof(argv[1]);
  ends = atof(argv[2]);
  fail_max = atoi(argv[3]);
  int64_t rp[2] = {0, 0};
  uint32_t dist[1];
  uint64_t far = 0;
  static char ws[65536] __attribute__((aligned(256)));
  const int rc = cldiam_sssp_delta_stepping(1, 0, rp, nullptr, 0, 1, dist, &far, ws, sizeof ws, nullptr);
  printf("status %d after %.0f s\n", rc, elapsed);
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    """A program that searches: first step at `begins` seconds, done at `ends`."""
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    d = str(tmp_path_factory.mktemp("host"))
    obj, src, exe = os.path.join(d, "sssp.o"), os.path.join(d, "runtime.cpp"), os.path.join(d, "search")
    subprocess.run(["hipcc", "-O1", "-fPIC", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-c",
                    os.path.join(CSRC, "sssp.hip"), "-o", obj], check=True)
    image = re.search(r"__hip_fatbin\w*", subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout)
    with open(src, "w") as f:
        f.write(RUNTIME)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which("hipcc"))))
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{rocm}/include", f"-I{os.path.join(CSRC, '..', '..', 'include')}",
                    src, obj, f"-Wl,--defsym={image.group(0)}=0", "-o", exe], check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout


def test_earlier_work_of_the_stream_is_not_the_search(search):
    assert "status 0 " in search(200, 205, 0)       # 200 s of other work, 5 of search
    assert "status 0 " in search(0, 50, 0)


def test_a_search_past_its_limit_ends(search):
    for begins in (0, 200):
        out = search(begins, begins + 10**6, 0)
        assert f"status {cd.CLDIAM_ETIMEOUT} " in out
        assert begins + 59 < float(out.split()[-2]) < begins + 63


def test_the_mirror_is_given_back_after_the_last_step(search):
    for out in (search(0, 3, 0), search(0, 3, 1), search(0, 10**6, 0)):
        assert "released with 0 steps queued" in out
    assert f"status {cd.CLDIAM_EHIP} " in search(0, 3, 1)       # a launch after the search fails
