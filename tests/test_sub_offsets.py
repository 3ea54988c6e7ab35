"""Where the sub-grid records of dense cells lie, from the functions that the
kernels use, compiled for the host: for every first point that a sort accepts,
the record starts inside the buffer, is found again from the cell's info, and
ends before the next one's."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_04514_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "device_common.h"
using namespace votess;
int64_t votess::sub_capacity(int64_t n) { return n / 2 + (20 * n) / 17 + 1024; }
int main(int argc, char** argv) {
  const int32_t* buffer = (const int32_t*)0x100000000000ull;
  const unsigned base = sub_base(atoll(argv[1]));
  for (int i = 2; i < argc; ++i) {
    const int b = (int)atoll(argv[i]);
    SubGrid s;
    s.start = buffer + base;
    const int2 info = make_int2(sub_offset(b, base), 1), none = make_int2(-1, 0);
    printf("%lld %d %d\n", (long long)(sub_record(s, info) - buffer), (int)is_dense(info), (int)is_dense(none));
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def positions(tmp_path_factory):
    d = tmp_path_factory.mktemp("sub")
    (d / "sub.hip").write_text(SRC)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1",
                    "-std=c++17", "-I", CSRC, str(d / "sub.hip"), "-o", str(d / "sub")], check=True,
                   capture_output=True)

    def run(n, bs):
        out = subprocess.run([str(d / "sub"), str(n), *map(str, bs)], check=True, capture_output=True, text=True).stdout
        rows = [tuple(map(int, line.split())) for line in out.splitlines()]
        assert all(dense == 1 and none == 0 for _, dense, none in rows)
        return [pos for pos, _, _ in rows]

    return run


@pytest.mark.parametrize("n,around", [(10_000, 0), (10 ** 7, 10 ** 6), (1_281_000_000, 1_280_990_000),
                                      (1_282_000_000, 0), (1_310_000_000, 1_303_800_000),
                                      (2 ** 31 - 2, 0), (2 ** 31 - 2, 1_304_000_000), (2 ** 31 - 2, 2 ** 31 - 2 - 4000)])
def test_records_lie_in_order_inside_the_buffer(positions, n, around):
    capacity = n // 2 + 20 * n // 17 + 1024
    bs = [around + i for i in range(0, 3000, 7)]
    at = dict(zip(bs, positions(n, bs)))
    assert all(p == 4 * (7 * b // 17) for b, p in at.items())
    lens = [17, 18, 19, 20, 21, 28, 35, 70, 350, 700]
    nxt = dict(zip([b + c for b in bs for c in lens], positions(n, [b + c for b in bs for c in lens])))
    for b in bs:
        for c in lens:
            words = (16 + c // 2 + 1 + 3) // 4 * 4
            assert 0 <= at[b] and at[b] + words <= nxt[b + c] and nxt[b + c] <= capacity
