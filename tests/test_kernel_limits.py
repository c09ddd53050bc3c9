"""Limits and choices of kernels, as the host code states them."""
import glob
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_03641_amd", "csrc")


def test_lds_limits_are_constants():
    """A kernel's limit of dynamic LDS holds for every handle of the process, so
    none sets it from its own sizes: a constant expression, no call or member of
    an object.  (A runtime that enforces the limit would refuse the launches of
    the handles with larger blocks; not every one does.)"""
    found = 0
    for f in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(f) as src:
            text = src.read()
        for m in re.finditer(r"hipFuncAttributeMaxDynamicSharedMemorySize,([^;]*);", text):
            value = re.sub(r"\((int|size_t)\)", "", m.group(1)).rstrip().rstrip(")")
            found += 1
            assert re.fullmatch(r"[\s\w:*+]+", value), (os.path.basename(f), value)
    assert found >= 2


def test_ilu_solve_choice(tmp_path):
    """The ILU solve stages its blocks in LDS only where that was measured to be
    the faster one: (rows, entries and levels of a block, blocks, us an
    application in LDS and in global memory)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no compiler")
    measured = [
        (16, 36, 16, 7053, 42.9, 22.2), (64, 190, 64, 14000, 232.8, 204.2), (48, 142, 47, 2351, 48.1, 40.5),
        (64, 346, 47, 1764, 44.1, 49.4), (128, 1004, 50, 882, 43.0, 67.2), (128, 656, 95, 6984, 220.2, 226.5),
        (128, 382, 127, 16511, 476.6, 438.4), (192, 574, 192, 417, 301.1, 137.8), (192, 1086, 111, 7383, 372.4, 359.5),
        (192, 1000, 127, 11008, 570.2, 640.9), (256, 1700, 97, 3492, 243.3, 307.2), (384, 3006, 101, 2328, 316.0, 301.2),
        (512, 4100, 72, 221, 61.7, 103.5), (512, 4040, 94, 1013, 159.2, 218.2), (512, 3850, 133, 4128, 983.1, 511.8),
        (768, 6400, 109, 1164, 444.8, 306.7), (1024, 8800, 103, 260, 160.2, 185.6), (1024, 8500, 145, 2064, 1114.7, 518.4),
    ]
    src, exe = tmp_path / "choice.cpp", str(tmp_path / "choice")
    rows = ",".join("{%d,%d,%d,%d}" % m[:4] for m in measured)
    src.write_text('#include <cstdio>\n#include "ilu.h"\nint main() {\n  const int m[][4] = {' + rows + '};\n'
                   '  for (auto &r : m) { vag::IluLds L; L.rows = r[0]; L.ents = r[1]; L.levs = r[2];'
                   ' std::printf("%d", (int)L.pays(r[3])); }\n}\n')
    inc = ["-I" + CSRC, "-I" + os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")]
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O0", "-w", *inc, str(src), "-o", exe],
                   check=True, capture_output=True)
    got = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    for m, g in zip(measured, got, strict=True):
        assert (g == "1") == (m[4] < m[5]), m


def test_estimates_admit_known_jobs():
    """A server refuses a job whose estimate exceeds its budget, so the estimates
    do not grow: bytes that admitted these jobs (cells a side, options, fracture
    faces) admit them."""
    import ctypes as C
    from paper_1602_03641_amd import vag
    amg, gmres, bicgstab = dict(precond=vag.VAG_PC_AMG), dict(krylov=vag.VAG_GMRES), dict(krylov=vag.VAG_BICGSTAB)
    mixed, ir = dict(precision=vag.VAG_MIXED), dict(precision=vag.VAG_MIXED_IR)
    for n, kw, nf, most in [(10, amg, 100, 21310981), (10, amg | mixed, 100, 21780666), (16, amg | mixed, 256, 34443621),
                            (16, amg, 0, 30772409), (24, amg | ir, 576, 72134810), (32, amg | mixed, 1024, 141396484),
                            (48, amg, 2304, 384072173), (48, amg | mixed | gmres, 2304, 644010186),
                            (64, amg | dict(amg_kind=1), 4096, 2575207893),
                            (48, bicgstab | dict(precond=vag.VAG_PC_BJILU0), 2304, 294023467),
                            (32, dict(precond=vag.VAG_PC_JACOBI), 1024, 73679915)]:
        o = vag.default_options(**kw)
        got = vag.load().vag_estimate_footprint((n + 1) ** 3, n ** 3, nf, C.byref(o))
        assert 0 < got <= most, (n, kw, got)


def _host_program(tmp_path, text, *args):
    """Compiles text against the library's headers (host code only) and returns
    what it prints."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no compiler")
    src, exe = tmp_path / "program.cpp", str(tmp_path / "program")
    src.write_text(text)
    inc = ["-I" + CSRC, "-I" + os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")]
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O0", "-w", *inc, str(src), *args, "-o",
                    exe], check=True, capture_output=True)
    return subprocess.run([exe], capture_output=True, text=True, check=True).stdout


def test_parts_are_not_tried_in_vain(tmp_path):
    """Calls that try to take their steps in parts of the mesh: every call of a
    handle whose parts fit; of one whose parts never fit, fewer and fewer, though
    never none; and every call again once they fit."""
    out = _host_program(tmp_path, """
#include <cstdio>
#include "vag_internal.h"
int main() {
    vag::HaloTries t;
    auto calls = [&](int n, bool fits) {
        int tried = 0;
        for (int k = 0; k < n; ++k)
            if (t.due()) ++tried, t.ended(false), fits ? t.ended(true) : void();
        return tried;
    };
    const int a = calls(50, true), b = calls(2, false), c = calls(998, false), d = calls(9000, false);
    std::printf("%d %d %d %d %d\\n", a, b, c, d, calls(256 + 100, true));
}
""")
    always, first, thousand, more, again = map(int, out.split())
    assert always == 50 and first == 1 and thousand <= 10
    assert 9000 // 256 <= more <= 9000 // 256 + 1
    assert again >= 100


def test_launches_of_many_rows(tmp_path):
    """The classical products take a wavefront per row.  A launch has fewer than
    2^32 threads, so rows from 2^26 on need several: every row once, none beyond
    (the library's launcher, with the runtime's launch replaced by a count)."""
    lib = os.path.join(os.path.dirname(CSRC), "libvag.so")
    if not os.path.exists(lib):
        pytest.skip("the library is not built")
    out = _host_program(tmp_path, """
#include <cstdio>
#include <cstdint>
#include "amg.h"
static dim3 grid, block;
static long long rows, next_row, bad;
extern "C" hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
    grid = g;
    block = b;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) {
    *g = grid;
    *b = block;
    *l = 0;
    *s = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void *, dim3 g, dim3 b, void **args, size_t, hipStream_t) {
    bad += (unsigned long long)g.x * b.x >= 1ull << 32 || *(int32_t *)args[0] != next_row;
    next_row += g.x;
    rows += (long long)g.x * g.y * g.z;
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
int main() {
    vag::Sell<double> A{};
    for (int n : {1, 1 << 20, (1 << 25) + 1, 1 << 26, (1 << 30) - 1})
        for (int k = 0; k < 4; ++k) {
            rows = next_row = 0;
            vag::cl_launch_product_rows(nullptr, n, k & 1 ? &A : nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                                        nullptr, nullptr, nullptr, k & 2, nullptr, nullptr, nullptr, nullptr);
            bad += rows != n;
        }
    std::printf("%lld\\n", bad);
}
""", "-rdynamic", "-x", "none", lib, "-Wl,-rpath," + os.path.dirname(lib))
    assert int(out) == 0


def test_polls_give_the_core_away(tmp_path):
    """A worker that waits for the device's rounds lets other threads have its
    core, and ends when the device has got there, or has nothing more to run."""
    out = _host_program(tmp_path, """
#include <cstdio>
#include "amg.h"
static int yields, queries, ends;
static volatile int started;
extern "C" int sched_yield() { return ++yields, 0; }
extern "C" hipError_t hipStreamQuery(hipStream_t) {
    if (++queries == 100) ends ? (void)0 : (void)(started = 5);
    return ends && queries > 100 ? hipSuccess : hipErrorNotReady;
}
int main() {
    for (ends = 0; ends < 2; ++ends) {
        yields = queries = started = 0;
        vag::poll_rounds(nullptr, &started, 3, 48);
        std::printf("%d %d %d\\n", yields, queries, started);
    }
}
""", "-rdynamic")
    begun, over = (tuple(map(int, line.split())) for line in out.splitlines())
    assert begun == (100, 100, 5) and over == (100, 101, 0)


def test_krylov_shape_choice(tmp_path):
    """Where the Krylov kernels go from four lanes per row to one: (unknowns, us
    of a solve with four, with one) of Jacobi CG and of CG with the aggregation
    hierarchy, the sizes at which both agree, and of BiCGStab."""
    lib = os.path.join(os.path.dirname(CSRC), "libvag.so")
    if not os.path.exists(lib):
        pytest.skip("the library is not built")
    cg = [(22707, 3396, 5274), (22707, 1911, 2380), (47915, 5789, 7585), (47915, 3386, 3815), (65559, 6137, 6219),
          (65559, 3831, 3960), (99405, 9083, 7358), (99405, 4460, 4211), (120000, 14878, 10668), (120000, 4635, 4229)]
    bcg = [(47915, 14258, 17321), (83160, 19100, 20700), (112847, 36756, 37143), (120000, 25400, 24000)]  # BiCGStab, Jacobi
    ilu = [(40425, 70700, 71700), (48159, 150400, 140800), (56700, 57700, 56000), (72000, 60100, 55700)]  # and ILU from global memory
    measured = [(m, line) for ms, line in ((cg, "kSplitMaxRows"), (bcg, "kSplitMaxBcg"), (ilu, "kSplitMaxIlu")) for m in ms]
    out = _host_program(tmp_path, """
#include <cstdio>
#include "vag_internal.h"
int main() {
    using namespace vag;
    const int64_t m[][2] = {%s};
    for (auto &r : m) std::printf("%%d ", (int)krylov_shape(r[0], r[1]).split);
}
""" % ",".join("{%d,%s}" % (m[0], line) for m, line in measured), "-x", "none", lib,
                        "-Wl,-rpath," + os.path.dirname(lib))
    for (m, line), g in zip(measured, out.split(), strict=True):
        assert (g == "1") == (m[1] < m[2]), (m, line)


def test_noalloc_operator_choice(tmp_path):
    """The allocation-free transport builds the upwind operator where that was
    measured to be faster: (cells a side, steps, us of a call with gathered
    steps, with the operator), where they differ by over 2 %."""
    measured = [(3, 10, 126, 130), (10, 8, 104, 123), (10, 16, 160, 144), (16, 8, 99, 121), (16, 12, 122, 137),
                (16, 18, 163, 152), (24, 10, 115, 123), (24, 12, 128, 131.9), (24, 16, 155, 143), (32, 8, 106, 117),
                (32, 12, 136, 127), (40, 4, 87, 107), (40, 10, 140, 132), (40, 12, 156, 141), (50, 4, 106, 118), (50, 6, 136, 130),
                (54, 4, 119, 134), (54, 5, 136, 141), (54, 6, 151, 146), (64, 2, 141, 166), (64, 4, 220, 182),
                (90, 4, 578, 385), (128, 4, 1623, 1030), (128, 8, 3030, 1225)]
    out = _host_program(tmp_path, """
#include <cstdio>
#include "vag_internal.h"
int main() {
    const int m[][2] = {%s};
    for (auto &r : m) {
        const long n = r[0];
        std::printf("%%d ", r[1] >= vag::noalloc_op_steps(n * n * n + (n + 1) * (n + 1) * (n + 1)));
    }
}
""" % ",".join("{%d,%d}" % m[:2] for m in measured))
    for m, g in zip(measured, out.split(), strict=True):
        assert abs(m[2] - m[3]) > 0.02 * m[2] and (g == "1") == (m[3] < m[2]), m
