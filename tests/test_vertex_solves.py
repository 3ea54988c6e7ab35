"""The solves of a vertex from three planes leave the compiler no choice of what
to fuse: taken from the kernel's source and built for the host with and without
contraction, they return the same bits."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLIP = os.path.join(ROOT, "paper_2412_04514_amd", "csrc", "clip.hip")

MAIN = r"""
int main() {
  double p[12];
  while (fread(p, 8, 12, stdin) == 12) {
    const V3<double> a = {p[0], p[1], p[2]}, b = {p[3], p[4], p[5]}, c = {p[6], p[7], p[8]};
    const V3<double> u = solve3<false>(a, p[9], b, p[10], c, p[11]), v = solve3<true>(a, p[9], b, p[10], c, p[11]);
    auto f = [](const V3<double>& x) -> V3<float> { return {(float)x.x, (float)x.y, (float)x.z}; };
    float err;
    const V3<float> w = solve3_err(f(a), (float)p[9], f(b), (float)p[10], f(c), (float)p[11], err);
    const double out[10] = {u.x, u.y, u.z, v.x, v.y, v.z, w.x, w.y, w.z, err};
    fwrite(out, 8, 10, stdout);
  }
  return 0;
}
"""


def _function(src, name):
    # from the line that begins the function (or its template) to its closing brace
    at = src.index(name + "(")
    start = src.rindex("\n\n", 0, at)
    return src[start:src.index("\n}\n", at) + 3]


def _build(d, contract):
    src = open(CLIP).read()
    v3 = "template <typename R>\nstruct V3 {\n  R x, y, z;\n};\n"
    assert v3 in src
    parts = [_function(src, "> solve3"), _function(src, "> solve3_err")]
    text = "#include <cfloat>\n#include <cmath>\n#include <cstdio>\n#include <hip/hip_runtime.h>\n" + v3
    text += "".join(parts).replace("__device__", "") + MAIN
    f = d / f"solve_{contract}.hip"
    f.write_text(text)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O3", "-mfma",
                    "-std=c++17", f"-ffp-contract={contract}", str(f), "-o", str(f.with_suffix(""))], check=True,
                   capture_output=True)
    return str(f.with_suffix(""))


@pytest.fixture(scope="module")
def solved(tmp_path_factory):
    d = tmp_path_factory.mktemp("solve")
    rng = np.random.default_rng(3)
    n = rng.standard_normal((50_000, 3, 3))
    c = 0.5 * (n ** 2).sum(axis=2) * rng.uniform(0.5, 2.0, (len(n), 3))
    x = np.concatenate([n.reshape(-1, 9), c], axis=1)
    out = {}
    for contract in ("fast", "off"):
        raw = subprocess.run([_build(d, contract)], input=x.tobytes(), check=True, capture_output=True).stdout
        out[contract] = np.frombuffer(raw).reshape(-1, 10)
    return n, c, out


def test_contraction_changes_no_bit(solved):
    _, _, out = solved
    assert out["fast"].shape == (50_000, 10)
    assert np.array_equal(out["fast"].view(np.int64), out["off"].view(np.int64))


def test_the_solves_solve(solved):
    n, c, out = solved
    want = np.linalg.solve(n, c[:, :, None])[:, :, 0]
    cond = np.linalg.cond(n)
    size = np.linalg.norm(want, axis=1)
    for k, eps in ((0, 2.0 ** -52), (3, 2.0 ** -52), (6, 2.0 ** -23)):
        err = np.linalg.norm(out["off"][:, k:k + 3] - want, axis=1)
        # Cramer's rule: each entry's products are off by a few ulps of their
        # sizes, which a condition number squared (two cross products) amplifies
        assert np.all(err <= 64 * eps * cond ** 2 * size)
