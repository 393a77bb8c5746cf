"""The split of a coarse SAP block over lane groups (coarse_sap_shape): for shapes
whose half sweep was timed with every number of parts, the one that the rule picks
is within a tenth of the fastest."""
import os
import re
import shutil
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1303_1377_amd", "csrc", "dd_coarse.hip")
CLANG = "/opt/rocm/llvm/bin/clang++"

# (bytes of a real, even sites, unknowns, RHS of a group, rows per load): us for 1, 2, ... parts
TIMED = {
    (8, 27, 32, 1, 1): [522.9, 509.2, 495.8, 480.4, 537.2, 505.8, 592.3],
    (8, 32, 24, 1, 1): [351.7, 344.2, 350.6, 333.0, 363.8, 421.0, 477.6, 346.2, 407.3],
    (8, 64, 4, 1, 1): [75.0, 54.3, 64.1, 75.7],
    (8, 64, 12, 1, 1): [195.7, 189.5, 237.2, 185.6, 223.5, 243.9, 294.7, 362.4],
    (4, 27, 16, 1, 2): [168.9, 97.4, 104.1, 79.8, 94.8, 102.0, 107.0, 111.3, 125.2, 131.9],
    (4, 27, 32, 1, 2): [365.2, 229.4, 273.3, 217.6, 252.2, 277.8, 313.5, 217.9, 235.1, 247.8],
    (4, 8, 40, 1, 2): [367.0, 208.4, 181.7, 159.9, 151.1, 151.9, 200.5, 199.3, 204.5, 156.3],
    (4, 64, 12, 1, 2): [143.1, 116.2, 112.1, 117.4, 134.5, 151.0, 163.7, 187.0, 197.4],
}


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    if not shutil.which(CLANG):
        pytest.skip("no " + CLANG)
    src = open(SRC).read()
    const = "".join(re.findall(r"^static constexpr (?:int CS_NT|int CS_PARTS|size_t CS_LDS) .*\n", src, re.M))
    cols = "".join(re.findall(r"^__host__ __device__ constexpr int coarse_sap_cols.*\n", src, re.M))
    start = src.index("struct SapShape {")
    body = src[start : src.index("\n}\n", src.index("coarse_sap_shape(int bv", start)) + 3]
    d = tmp_path_factory.mktemp("sap_shape")
    (d / "m.cpp").write_text("""#include <algorithm>
#include <cstdio>
#include <cstdlib>
#define __host__
#define __device__
template <class T> struct cx { T re, im; };
%s%s%s
template <class T> void refused() {
    for (int nd = 2; nd <= 64; nd += 2)
        for (int bv = 1; bv * nd <= 2048; bv++)
            for (int rpl = 1; rpl <= 4; rpl *= 2) {
                if (nd %% rpl || (sizeof(T) == 8 && rpl > 1)) continue;
                const SapShape s = coarse_sap_shape<T>(bv, nd, 1, rpl), b = coarse_sap_shape<T>(bv, nd, 1, rpl, true);
                const SapShape& c = s.ok ? s : b;
                if (!c.ok || c.lds > 160 * 1024 || c.parts < 1 || c.hops < 1 || (long)c.nt * c.nv < (long)bv * nd) printf("%%d x %%d ", bv, nd);
            }
}
int main(int n, char** a) {
    if (n == 1) {
        refused<double>();
        refused<float>();
        return 0;
    }
    const int bv = atoi(a[2]), nd = atoi(a[3]), kr = atoi(a[4]), rpl = atoi(a[5]);
    const SapShape s = atoi(a[1]) == 8 ? coarse_sap_shape<double>(bv, nd, kr, rpl) : coarse_sap_shape<float>(bv, nd, kr, rpl);
    printf("%%d", s.ok ? s.parts : 0);
}
""" % (const, cols, body))
    exe = str(d / "m")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-o", exe, str(d / "m.cpp")], check=True)
    return lambda *shape: subprocess.run([exe, *map(str, shape)], check=True, capture_output=True, text=True).stdout


@pytest.mark.parametrize("shape", list(TIMED), ids=str)
def test_parts(parts, shape):
    p, us = int(parts(*shape)), TIMED[shape]
    assert 1 <= p <= len(us)
    assert us[p - 1] <= 1.1 * min(us), "%d parts: %.1f us, the fastest takes %.1f" % (p, us[p - 1], min(us))


def test_every_admitted_block_has_a_shape(parts):
    """configure admits blocks of up to 2048 rows of one parity."""
    assert parts() == ""
