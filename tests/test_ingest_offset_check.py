"""The ingest's check of the row offsets has to cost a few accesses per row
whatever the offsets hold: it meets the malformed ones.  Its kernel is run here
on the CPU, thread by thread, with counted accesses; the GPU test refuses
offsets that alternate between the ends of the arcs."""
import os
import re
import subprocess

import numpy as np
import pytest

import graphgen
import paper_1506_03265_amd as cd

SOURCE = os.path.join(os.path.dirname(os.path.abspath(cd.__file__)), "csrc", "ingest.hip")

HARNESS = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>
static long accesses, limit;
template <class T> struct Counted {   // an array whose accesses are counted
  T *p;
  T &operator[](int64_t i) const { if (++accesses > limit) { puts("too many accesses"); exit(3); } return p[i]; }
};
struct Dim { unsigned x = 0; };
static Dim blockIdx, threadIdx, blockDim, gridDim;
enum : uint32_t { BAD_ROWPTR = 1 };
constexpr int kTile = 2048;
struct IngestCtl { uint32_t bad; };
static uint32_t atomicOr(uint32_t *p, uint32_t x) { uint32_t y = *p; *p |= x; return y; }
@KERNEL@
int main(int argc, char **argv) {
  const int32_t n = atoi(argv[1]);
  const int64_t m = atoll(argv[2]);
  const bool alternate = atoi(argv[3]) != 0;
  std::vector<int64_t> offsets(n + 1);
  for (int64_t i = 0; i <= n; ++i) offsets[i] = alternate ? (i & 1) * m : i * m / n;
  std::vector<int32_t> notes(m / kTile + 2);
  IngestCtl c{0};
  limit = 8 * (long)n + 2 * (m / kTile) + 64;
  Counted<const int64_t> rp{offsets.data()};
  Counted<int32_t> tile_row{notes.data()};
  IngestCtl *ctl = &c;
  blockDim.x = 256;
  gridDim.x = 16;
  for (blockIdx.x = 0; blockIdx.x < gridDim.x; ++blockIdx.x)
    for (threadIdx.x = 0; threadIdx.x < blockDim.x; ++threadIdx.x) k_check_rows(@ARGS@);
  printf("%u\n", c.bad);
  (void)tile_row;
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    """A program that runs k_check_rows over n rows of m arcs and prints the flags."""
    text = open(SOURCE).read()
    found = re.search(r"__global__ void __launch_bounds__\(kT\) (k_check_rows\(([^)]*)\) \{.*?\n\})", text, re.S)
    params = [p.split()[-1].lstrip("*") for p in found.group(2).split(",")]
    body = re.sub(r"const int64_t \*rp", "Counted<const int64_t> rp", found.group(1))
    body = re.sub(r"int32_t \*tile_row", "Counted<int32_t> tile_row", body)
    d = tmp_path_factory.mktemp("check")
    (d / "check.cpp").write_text(HARNESS.replace("@KERNEL@", "static void " + body).replace("@ARGS@", ", ".join(params)))
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(d / "check"), str(d / "check.cpp")], check=True)
    return lambda n, m, alternate: subprocess.run([str(d / "check"), str(n), str(m), str(int(alternate))],
                                                  capture_output=True, text=True, timeout=60)


@pytest.mark.parametrize("n,m", [(1001, 4096), (20000, 4_000_000), (100000, 300_000_000)])
def test_work_of_the_check_is_linear(check, n, m):
    run = check(n, m, False)
    assert run.returncode == 0 and run.stdout.split() == ["0"]
    run = check(n, m, True)
    assert run.returncode == 0, run.stdout
    assert run.stdout.split() == ["1"]


@pytest.mark.gpu
def test_alternating_offsets_are_refused():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, m = 4000, 40960
    rng = np.random.default_rng(1)
    col, w = rng.integers(0, n, m).astype(np.int32), np.ones(m, np.uint32)
    for last in (m, 0):
        rp = np.where(np.arange(n + 1) % 2 == (0 if last == 0 else n % 2), last, m - last).astype(np.int64)
        rp[0] = 0
        print(f"[ingest] offsets alternating, the last one {rp[-1]}", flush=True)
        with pytest.raises(cd.CldiamError) as e:
            cd.cldiam_load_csr(graphgen.Graph(n, rp, col, w))
        assert e.value.status == cd.CLDIAM_EINVAL and "row offsets" in str(e.value)
