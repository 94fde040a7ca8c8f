"""Host-only check of the fp64 normal distribution of the fp32 row kernels (csrc/common.hip.h): the table's evaluation and the
arithmetic around it are compiled with the host compiler and compared with 40-digit values over the whole range that does not
underflow.

Bounds, relative, u = 2^-53: Phi(-a) is a node (one rounding), what lies between it and a (a tenth of it at most, so that its own
few roundings count as one) and their difference (one): 4 u, and 45 w (h^2)^2 / 322560 with w = (13.25 / 128)^2, h = 1/128, of that
tenth, the largest term left out: 6e-16 more.  phi is a node and a factor within 11 % of one: 3 u.  Beyond the table an exponential
and three products: 5 u.  The library calls that the table stands in for are within 3e-14 and 2.6e-16."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2509_14279_amd", "csrc", "common.hip.h")
U = 2.0 ** -53


@pytest.fixture(scope="module")
def values(tmp_path_factory):
    text = open(HEADER).read()
    code = text[text.index("namespace ctmath {\n// Sums and products"):text.index("struct NormalTable {")]
    code = code.replace("__device__ const NormalTableData", "static const NormalTableData").replace('"+s"', '"+r"')
    prog = ("#include <cmath>\n#include <cstdio>\n#include <initializer_list>\n#define __device__\n#define __forceinline__ inline\nusing std::exp;\n" + code +
            """int main() {
  for (int i = 0; i < 20000; i++) {
    // fp32 numbers: spread evenly, and around the nodes and the places half way between them
    const double even = (double)(float)(i * (38.0 / 20000)), k = std::nearbyint(even * 128) / 128;
    const float near = (float)k;
    const double all[4] = {even, (double)near, (double)std::nextafterf(near, 99.0f), (double)std::nextafterf(near, 0.0f)};
    for (double z : all) {
      double q, phi;
      if (z > 13.25) normal_tail<true>(z, q, phi);
      else {
        const int n = (int)std::nearbyint(z * 64);
        normal_near<true>(z, z - n / 64.0, g_normal_table.node[n].tail, g_normal_table.node[n].density, q, phi);
      }
      std::printf("%a %a %a\\n", z, q, phi);
    }
  }
  for (double z : {40.0, 51.9, 52.1, 1e3, 1e8, 1e10, 1e15, 1e20, 1e25, 1e30, 1e38, (double)__FLT_MAX__, (double)INFINITY}) {
    double q, phi;
    normal_tail<true>(z, q, phi);
    std::printf("%a %a %a\\n", z, q, phi);
  }
}
""")
    d = tmp_path_factory.mktemp("normal")
    src, exe = d / "normal.cpp", d / "normal"
    src.write_text(prog)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    v = [float.fromhex(x) for x in out]
    return sorted(set(zip(v[0::3], v[1::3], v[2::3])))


def test_tail_and_density(values):
    mp = pytest.importorskip("mpmath")
    mp.mp.dps = 40
    for z, q, phi in values[::5]:
        if z >= 40:
            continue
        x = mp.mpf(z)
        exact, density = mp.erfc(x / mp.sqrt(2)) / 2, mp.exp(-x * x / 2) / mp.sqrt(2 * mp.pi)
        if density < mp.mpf(2) ** -1000:
            continue
        assert abs(q / exact - 1) <= (5 * U if z > 13.25 else 4 * U + 6e-16), z
        assert abs(phi / density - 1) <= (5 * U if z > 13.25 else 3 * U), z


def test_beyond_the_smallest_double(values):
    # both are zero there, at the largest fp32 number and at infinity as well: Phi is exactly 0 or 1
    beyond = [v for v in values if v[0] >= 40]
    assert beyond[-1][0] == float("inf") and len(beyond) == 13
    for z, q, phi in beyond:
        assert q == 0 and phi == 0, (z, q, phi)
