"""CPU check of the inflow speed's root: the kernel's own function, compiled for the host from the
kernel source, gives the bits of the 60 bisections that define the root, over the distribution's
bulk and far into both tails (uniform draws never reach the lower one)."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _function(src, head):
    """The text of the function that starts with `head`."""
    at = src.index(head)
    depth, i = 0, src.index("{", at)
    while True:
        depth += {"{": 1, "}": -1}.get(src[i], 0)
        i += 1
        if depth == 0:
            return src[at:i]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    src = open(os.path.join(ROOT, "paper_2007_13091_amd", "csrc", "kernels.hip")).read()
    parts = [_function(src, "__device__ __forceinline__ double npdf("), _function(src, "__device__ __forceinline__ double ncdf("),
             _function(src, "__device__ double flux_speed(")]
    pi = re.search(r"constexpr double kPi = [^;]*;", open(os.path.join(
        ROOT, "paper_2007_13091_amd", "csrc", "device_common.hpp")).read() + src).group(0)
    code = "#include <cmath>\nusing std::fabs; using std::fmin; using std::sqrt; using std::exp; using std::erfc;\n" + pi + "\n"
    code += "\n".join(parts) + """
static double bisect(double a, double eta) {
    const double pa = npdf(a), Z = pa + a * ncdf(a), cm = ncdf(-a);
    double lo = 0.0, hi = (a > 0.0 ? a : 0.0) + 40.0;
    for (int it = 0; it < 60; ++it) {
        const double z = 0.5 * (lo + hi);
        const double G = (pa - npdf(z - a) + a * (ncdf(z - a) - cm)) / Z;
        if (G < eta) lo = z; else hi = z;
    }
    return 0.5 * (lo + hi);
}
extern "C" void both(long n, const double *a, const double *eta, double *fast, double *plain) {
    for (long i = 0; i < n; ++i) { fast[i] = flux_speed(a[i], eta[i]); plain[i] = bisect(a[i], eta[i]); }
}
"""
    d = tmp_path_factory.mktemp("speed")
    (d / "speed.cpp").write_text(code)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-D__device__=",
                    "-D__forceinline__=inline", "-o", str(d / "speed.so"), str(d / "speed.cpp")], check=True)
    lib = C.CDLL(str(d / "speed.so"))
    p = np.ctypeslib.ndpointer(np.float64, flags="C")
    lib.both.argtypes = [C.c_long, p, p, p, p]
    return lib


@pytest.mark.parametrize("draws", ["uniform", "low tail", "high tail"])
@pytest.mark.parametrize("a_range", [(-5.0, -2.9), (-3.0, -1.0), (-1.0, 0.5), (0.5, 5.0), (5.0, 40.0), (40.0, 300.0)])
def test_speed_is_the_bisections_root_to_the_bit(host, a_range, draws):
    rng = np.random.default_rng([int(10 * (a_range[1] + 10)), len(draws)])
    n = 60000
    a = rng.uniform(*a_range, n)
    tail = 10.0 ** rng.uniform(-15.0, -1.0, n)
    eta = {"uniform": (rng.integers(0, 2 ** 52, n) + 0.5) * 2.0 ** -52, "low tail": tail, "high tail": 1.0 - tail}[draws]
    fast, plain = np.empty(n), np.empty(n)
    host.both(n, a, eta, fast, plain)
    same = (fast == plain) | (np.isnan(fast) & np.isnan(plain))
    assert same.all(), (int((~same).sum()), a[~same][:3], eta[~same][:3], np.abs(fast - plain)[~same].max())
