"""The index that a thread of the small-cell pass takes, from the kernel's own
function compiled for the host: each cell once, and nothing past the last one,
up to grids that end just below 2^31 cells."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_04514_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "device_common.h"
int main(int, char** argv) {
  const int count = atoi(argv[1]), threads = 1024;
  const unsigned last = (unsigned)(((long long)count + threads - 1) / threads) - 1u;
  for (unsigned b = last > 1 ? last - 1 : 0; b <= last; ++b)
    for (unsigned t = 0; t < (unsigned)threads; ++t) printf("%d\n", votess::thread_item(b, threads, t, count));
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("items")
    (d / "items.hip").write_text(SRC)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1",
                    "-std=c++17", "-I", CSRC, str(d / "items.hip"), "-o", str(d / "items")], check=True,
                   capture_output=True)
    return str(d / "items")


@pytest.mark.parametrize("count", [1, 1023, 1024, 1025, 2 ** 31 - 1025, 2 ** 31 - 1024, 2 ** 31 - 1023, 2 ** 31 - 300,
                                   2 ** 31 - 2])
def test_threads_take_each_cell_once(program, count):
    out = subprocess.run([program, str(count)], check=True, capture_output=True, text=True).stdout
    got = [int(x) for x in out.split()]
    first = max(0, -(-count // 1024) - 2) * 1024
    assert got == [min(first + i, count) for i in range(len(got))]
    assert got[-1] >= count - 1
