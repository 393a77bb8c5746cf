"""The first kernel of a coarsest-level Arnoldi step runs beside the workgroup
that folds the step before and may raise the stop flag, so the waves of one
workgroup can read the flag before and after it changes.  Both vector-unit forms
of that kernel are run on the CPU, lane by lane, with the flag changed between
the first wave and the others, both ways round: the workgroup must do the whole
of its work or none of it (half of it reads input pointers that were never
stored)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1303_1377_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

# One workgroup on one thread: every lane is a context that runs to its next
# workgroup barrier or lane exchange; lanes that have returned count as arrived.
SHIM = r"""
#pragma once
#include <math.h>
#include <stddef.h>
#include <string.h>
#include <ucontext.h>
#include <functional>
#include <vector>
#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
typedef void* hipStream_t;
typedef int hipError_t;
inline dim3 threadIdx, blockIdx, blockDim, gridDim;
template <class T> T min(T a, T b) { return a < b ? a : b; }
template <class T> T max(T a, T b) { return a > b ? a : b; }
namespace emu {
enum { RUN, WAVE, GROUP, DONE };
struct Lane { ucontext_t c; std::vector<char> stack; int state; long long val; };
inline std::vector<Lane> lanes;
inline ucontext_t home;
inline int cur;
inline std::function<void()> body;
inline void wait(int s) { lanes[cur].state = s; swapcontext(&lanes[cur].c, &home); }
inline void entry() { body(); lanes[cur].state = DONE; }
inline void release(int a, int b, int s) { for (int i = a; i < b; i++) if (lanes[i].state == s) lanes[i].state = RUN; }
inline void run_wave(int w) {   // until each of its lanes has returned or waits at a workgroup barrier
    for (;;) {
        bool ran = false;
        for (int i = 64 * w; i < 64 * w + 64; i++)
            if (lanes[i].state == RUN) { ran = true; cur = i; threadIdx.x = i; swapcontext(&home, &lanes[i].c); }
        if (!ran) {
            bool any = false;
            for (int i = 64 * w; i < 64 * w + 64; i++) any = any || lanes[i].state == WAVE;
            if (!any) return;
            release(64 * w, 64 * w + 64, WAVE);
        }
    }
}
// waves in `order`; between() runs after the first of them has reached its first barrier
inline void group(int waves, const std::vector<int>& order, std::function<void()> between, std::function<void()> f) {
    body = f;
    lanes.assign(64 * waves, Lane());
    blockDim = dim3(64 * waves);
    for (auto& l : lanes) {
        l.stack.resize(1 << 16);
        getcontext(&l.c);
        l.c.uc_stack.ss_sp = l.stack.data();
        l.c.uc_stack.ss_size = l.stack.size();
        l.c.uc_link = &home;
        makecontext(&l.c, entry, 0);
    }
    for (bool first = true, live = true; live; first = false) {
        for (size_t o = 0; o < order.size(); o++) { run_wave(order[o]); if (first && o == 0) between(); }
        live = false;
        for (auto& l : lanes) live = live || l.state == GROUP;
        release(0, 64 * waves, GROUP);
    }
}
template <class T> T from_lane(T v, int src) {   // v of lane src of the wave
    lanes[cur].val = 0;
    memcpy(&lanes[cur].val, &v, sizeof v);
    wait(WAVE);
    memcpy(&v, &lanes[(cur & ~63) + src].val, sizeof v);
    wait(WAVE);
    return v;
}
inline int dpp(int v, int ctrl) {
    const int l = cur & 63;
    return from_lane(v, ctrl == 0xB1 ? l ^ 1 : ctrl == 0x4E ? l ^ 2 : ctrl == 0x141 ? l ^ 7 : l ^ 15);
}
}  // namespace emu
inline void __syncthreads() { emu::wait(emu::GROUP); }
template <class T> T __shfl_xor(T v, int m, int) { return emu::from_lane(v, (emu::cur & 63) ^ m); }
#define __builtin_amdgcn_mov_dpp(v, ctrl, ...) emu::dpp(v, ctrl)
#define __builtin_amdgcn_readlane(v, l) emu::from_lane((int)(v), l)
#define __builtin_amdgcn_readfirstlane(v) emu::from_lane((int)(v), 0)
struct Swap2 { unsigned v[2]; unsigned operator[](int i) const { return v[i]; } };
#define __builtin_amdgcn_permlane32_swap(a, b, ...) Swap2{{a, b}}
#define __builtin_amdgcn_permlane16_swap(a, b, ...) Swap2{{a, b}}
template <class D, class S> D bits(S s) { D d; memcpy(&d, &s, sizeof d); return d; }
inline int __float_as_int(float f) { return bits<int>(f); }
inline float __int_as_float(int i) { return bits<float>(i); }
inline long long __double_as_longlong(double d) { return bits<long long>(d); }
inline double __longlong_as_double(long long i) { return bits<double>(i); }
"""

MAIN = r"""
#include "dd_gmres.h"
#include <stdio.h>
#include <stdlib.h>
#include <vector>
namespace dd {
%s
}
using namespace dd;
typedef cx<double> Z;
int main(int argc, char** argv) {
    const bool rows = atoi(argv[1]);
    const int flag0 = atoi(argv[2]);   // the stop flag until the first wave has run; then the other value
    const int nd = 20, vh = 8;
    Geom g{};
    for (int mu = 0; mu < 4; mu++) { g.d[mu] = g.b[mu] = 2; g.lb[mu] = 1; g.nb[mu] = 1; }
    g.bvh = g.vh = vh; g.lbvh = 3; g.nblk = 1;
    auto fill = [](size_t n, unsigned s) {
        std::vector<Z> v(n);
        for (auto& z : v) { s = s * 1664525u + 1013904223u; z.re = (s >> 8) / 1e7 - 0.8; z.im = (s >> 20) / 4e3 - 0.5; }
        return v;
    };
    const auto M = fill((size_t)2 * vh * 9 * nd * nd, 1), Minv = fill((size_t)2 * vh * nd * nd, 2), in = fill(2 * vh * nd, 3);
    CoarseOp<double> op{g, nd, M.data(), Minv.data()};
    const Z npart[2] = {{1.5, 0}, {2.5, 0}};
    static GmDev st;
    InScale isc{&st, 1, 2, npart, 2, npart, 0};
    const Mask live{&st.stop, 1, 1};
    constexpr int rc = 128 / (int)sizeof(Z), nrc = (nd + rc - 1) / rc;
    const int waves = rows ? 4 : 3;
    auto pass = [&](int first, bool flip, std::vector<int> order) {
        std::vector<Z> out(2 * vh * nd, Z{-7, -7});
        st.stop = first;
        blockIdx = dim3(rows ? 5 * nrc : 5, 0);   // site 5 (its first rows)
        emu::group(waves, order, [&] { if (flip) st.stop = !st.stop; }, [&] {
            if (rows) k_coarse_rows<double, double, rc>(op, 0, CS_NONE, nullptr, 1, 0, in.data(), out.data(), live, 0, isc, vh * nrc);
            else k_coarse_apply<double, double>(op, 0, CS_NONE, nullptr, 1, in.data(), 1, out.data(), live, 0, isc, vh);
        });
        return out;
    };
    std::vector<int> up, down;
    for (int w = 0; w < waves; w++) { up.push_back(w); down.push_back(waves - 1 - w); }
    auto same = [](const std::vector<Z>& a, const std::vector<Z>& b) { return !memcmp(a.data(), b.data(), sizeof(Z) * a.size()); };
    const bool back = atoi(argv[3]);
    const auto got = pass(flag0, true, back ? down : up);
    const auto all = pass(0, false, up), none = std::vector<Z>(2 * vh * nd, Z{-7, -7});
    if (same(all, none)) return 3;
    printf("%%s\n", same(got, all) ? "all" : same(got, none) ? "none" : "part");
    return 0;
}
"""


def _kernel(src, name):
    """The text of a kernel template of the source, from its template line to its closing brace."""
    at = src.index(" " + name + "(CoarseOp")
    start = src.rindex("\ntemplate <", 0, at)
    return src[start : src.index("\n}\n", at) + 3]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which(CLANG):
        pytest.skip("no " + CLANG)
    d = tmp_path_factory.mktemp("stop_flag")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(SHIM)
    src = open(os.path.join(CSRC, "dd_coarse.hip")).read()
    pre = src[src.index("static constexpr int CA_WAVES") : src.index("};", src.index("struct CaPre")) + 3]
    (d / "main.cpp").write_text(MAIN % (pre + _kernel(src, "k_coarse_apply") + _kernel(src, "k_coarse_rows")))
    exe = str(d / "stop_flag")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-I", str(d), "-I", CSRC, "-o", exe, str(d / "main.cpp")], check=True)
    return exe


@pytest.mark.parametrize("order", ["first wave first", "first wave last"])
@pytest.mark.parametrize("flag", [0, 1])
@pytest.mark.parametrize("kernel", ["apply", "rows"])
def test_waves_that_disagree(program, kernel, flag, order):
    r = subprocess.run([program, "1" if kernel == "rows" else "0", str(flag), "1" if "last" in order else "0"],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, "the kernel ended with status %d" % r.returncode
    assert r.stdout.strip() in ("all", "none")
