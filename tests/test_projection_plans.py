"""Properties of the projection plans (host arithmetic, compiled and run on the CPU)."""
import os
import shutil
import subprocess
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_13144_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")

HEAD = textwrap.dedent(r"""
    #include <cstdio>
    #include <cstring>
    #include <initializer_list>
    #include "ss_plan.h"
    static inline bool same(const ss::GemmPlan& a, const ss::GemmPlan& b) { return std::memcmp(&a, &b, sizeof a) == 0; }   // ints only
    struct Mat { int N, Kp, epi, max_ksplit; };
    // q|k|v, o, gate|up, down and the head of models of every width the library takes
    template <class F> static int every_matrix(F f) {
        const int dims[] = {64, 256, 512, 1024, 2048, 3072, 4096, 5120, 8192};
        const int ffns[] = {16, 688, 2752, 11008, 13824, 28672};
        for (int d : dims)
            for (int F_ : ffns) {
                const int Fp = (F_ + 63) / 64 * 64;
                const Mat mats[] = {{3 * d, d, ss::EPI_PARTIAL, 8}, {d, d, ss::EPI_PARTIAL, 8}, {2 * F_, d, ss::EPI_SWIGLU, 8},
                                    {d, Fp, ss::EPI_PARTIAL, 8}, {32000, d, ss::EPI_PARTIAL, 1}, {1040, d, ss::EPI_PARTIAL, 1}};
                for (const Mat& m : mats)
                    if (int rc = f(m)) return rc;
            }
        return 0;
    }
""")


def _run(tmp_path, body):
    drv = tmp_path / "driver.cpp"
    drv.write_text(HEAD + textwrap.dedent(body))
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-I", CSRC, str(drv), os.path.join(CSRC, "ss_plan.cpp"), "-o", str(exe)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_row_counts_of_one_strip_share_a_plan(tmp_path):
    """A micro-batch that shrinks keeps its launch shapes until it has lost a whole strip of 16 rows: its rows' numbers stay
    the same, bit for bit, until then."""
    _run(tmp_path, r"""
        int main() {
            return every_matrix([](const Mat& m) {
                for (int cu : {64, 256, 304})
                    for (int n = 1; n <= 1040; ++n) {
                        const int full = (n + 15) / 16 * 16;
                        if (same(ss::gemm_plan(m.N, m.Kp, n, m.epi, cu, m.max_ksplit), ss::gemm_plan(m.N, m.Kp, full, m.epi, cu, m.max_ksplit)))
                            continue;
                        std::printf("N %d Kp %d epilogue %d cu %d: %d and %d rows differ\n", m.N, m.Kp, m.epi, cu, n, full);
                        return 1;
                    }
                return 0;
            });
        }
    """)
