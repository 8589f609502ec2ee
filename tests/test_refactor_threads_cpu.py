"""The value check of a numeric re-setup (Sec. V-A) where no thread can be
started: it takes all the values itself.  Built here with the host sources and a
pthread_create that always fails (a process at its thread limit)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_04876_amd", "csrc")

MAIN = r"""
#include <cerrno>
#include <cstdio>
#include <limits>
#include <vector>
#include <pthread.h>
#include "gdsw_impl.hpp"
extern "C" int pthread_create(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *) { return EAGAIN; }
extern "C" void gdsw_default_options(gdsw_options *) {}   // (the C entry's, not used here)
int main() {
    for (long n : {0L, 1L, 799999L, 800000L, 3000001L}) {
        std::vector<double> v(n, 1.0);
        if (!gdsw::all_finite(v.data(), n)) return 1;
        for (long p : {0L, n / 8, n / 2, n - 1}) {
            if (p < 0 || p >= n) continue;
            v[p] = std::numeric_limits<double>::infinity();
            if (gdsw::all_finite(v.data(), n)) return 2;
            v[p] = 1.0;
        }
    }
    std::puts("ok");
}
"""


def test_value_check_without_threads(tmp_path):
    main = tmp_path / "main.cpp"
    main.write_text(MAIN)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-O0", "-std=c++17", "-fopenmp", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    str(main), os.path.join(CSRC, "symbolic.cpp"), os.path.join(CSRC, "nd.cpp"), "-o", exe, "-lpthread"],
                   check=True, capture_output=True, timeout=300)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", (out.returncode, out.stderr)
