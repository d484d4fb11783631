"""The host loop of the decomposition against a stand-in for the GPU, on the CPU:
its host code is linked with a small runtime whose stream runs the launched
sweeps only when the host waits for it.  The mapped buffer that queued sweeps
write is not given back before they have run, whichever call fails."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1506_03265_amd as cd

CSRC = os.path.join(os.path.dirname(os.path.abspath(cd.__file__)), "csrc")

RUNTIME = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include "cldiam.h"

static std::map<const void *, std::string> names;
static char buffer[4096] __attribute__((aligned(256)));   // the pooled one
static int queued = 0, launched = 0;   // sweeps on the stream, sweeps in all
static int bad_sweep = 0;              // the launch of this sweep fails
static int bad_record = 0, records = 0;   // this event record fails
static hipError_t error = hipSuccess;

extern "C" {
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *name, const char *, unsigned, void *, void *, void *, void *, int *) {
  names[f] = name;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t) {
  if (names[f].find("k_sweep") == std::string::npos) return hipSuccess;
  ++queued;
  // the device reports progress and, with the 40th sweep, the end
  volatile uint32_t *mirror = (volatile uint32_t *)(buffer + sizeof buffer - 128);
  mirror[0] = ++launched > 8 ? launched - 8 : 0;
  if (launched >= 40) mirror[1] = 1;
  if (launched == bad_sweep) error = hipErrorLaunchFailure;
  return error;
}
hipError_t hipLaunchCooperativeKernel(const void *, dim3, dim3, void **, unsigned, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = error; error = hipSuccess; return e; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { queued = 0; return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyDeviceToHost) { queued = 0; memset(to, 0, n); }
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return ++records == bad_record ? hipErrorUnknown : hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
hipError_t hipHostMalloc(void **, size_t, unsigned) { abort(); }
hipError_t hipHostFree(void *) { abort(); }
const char *cldiam_strerror(int) { return ""; }
}
namespace cld {
void set_error(const char *, ...) {}
int hip_fail(hipError_t, const char *) { return CLDIAM_EHIP; }
void *pinned_acquire(size_t) { return buffer; }
void pinned_release(void *) { printf("released with %d sweeps queued\n", queued); }
int cooperative_blocks(const void *, int, int, int *blocks) { *blocks = 256; return CLDIAM_OK; }
}

int main(int argc, char **argv) {
  bad_sweep = atoi(argv[1]);
  bad_record = atoi(argv[2]);
  static int64_t rp[3] = {0, 0, 0};
  static uint64_t arcs[1];
  static int32_t cluster[2];
  static uint64_t dist[2];
  static char ws[1 << 22] __attribute__((aligned(256)));
  cldiam_graph g;
  memset(&g, 0, sizeof g);
  g.n = 2;
  g.d_row_ptr = rp;
  g.d_arcs = arcs;
  g.d_cluster = cluster;
  g.d_D = dist;
  g.params.tau = 1;
  cldiam_stats st;
  const int rc = cldiam_decompose(&g, &st, CLDIAM_DRIVER_HOST, nullptr, ws, sizeof ws, nullptr);
  printf("status %d after %d sweeps\n", rc, launched);
}
"""


@pytest.fixture(scope="module")
def job(tmp_path_factory):
    """A program that decomposes: one sweep's launch, or one event record, fails."""
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    d = str(tmp_path_factory.mktemp("host"))
    obj, src, exe = os.path.join(d, "decompose.o"), os.path.join(d, "runtime.cpp"), os.path.join(d, "job")
    subprocess.run(["hipcc", "-O1", "-fPIC", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-c",
                    os.path.join(CSRC, "decompose.hip"), "-o", obj], check=True)
    image = re.search(r"__hip_fatbin\w*", subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout)
    with open(src, "w") as f:
        f.write(RUNTIME)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which("hipcc"))))
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{rocm}/include", f"-I{os.path.join(CSRC, '..', '..', 'include')}",
                    src, obj, f"-Wl,--defsym={image.group(0)}=0", "-o", exe], check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout


@pytest.mark.parametrize("sweep,record", [(0, 0), (16, 0), (40, 0), (0, 2)])
def test_the_mirror_is_given_back_after_the_last_sweep(job, sweep, record):
    out = job(sweep, record)
    assert "released with 0 sweeps queued" in out
    assert int(out.split()[-2]) >= 16
    if sweep or record:
        assert f"status {cd.CLDIAM_EHIP} " in out
