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
    // q|k|v, o, gate|up, down and the head of models of every width the library takes, q|k|v, o and down with every
    // epilogue that they are planned with
    template <class F> static int every_matrix(F f) {
        const int dims[] = {64, 256, 512, 1024, 2048, 3072, 4096, 5120, 8192};
        const int ffns[] = {16, 688, 2752, 11008, 13824, 28672};
        for (int d : dims)
            for (int F_ : ffns) {
                const int Fp = (F_ + 63) / 64 * 64;
                const Mat mats[] = {{3 * d, d, ss::EPI_PARTIAL, 8}, {3 * d, d, ss::EPI_QKV, 8}, {d, d, ss::EPI_PARTIAL, 8}, {d, d, ss::EPI_RESIDUAL, 8},
                                    {2 * F_, d, ss::EPI_SWIGLU, 8}, {d, Fp, ss::EPI_PARTIAL, 8}, {d, Fp, ss::EPI_RESIDUAL, 8}, {32000, d, ss::EPI_PARTIAL, 1}, {1040, d, ss::EPI_PARTIAL, 1}};
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
                    for (int n = 1; n <= 12320; n += n <= 1040 ? 1 : 7) {
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


def test_kernel_choice_follows_the_measurements(tmp_path):
    """Sweep or block kernel at 145 to 256 rows, on 256 compute units, wherever one of them was measured 4 % faster or more."""
    _run(tmp_path, r"""
        struct Point { int N, Kp, epi, max_ksplit, rows; bool sweep; };
        int main() {
            const int P = ss::EPI_PARTIAL, S = ss::EPI_SWIGLU;
            const Point points[] = {
                // d 4096, ffn 11008: q|k|v, gate|up, head (us, sweep / block)
                {12288, 4096, P, 8, 160, true},     // 32.7 / 34.8
                {22016, 4096, S, 8, 160, true},     // 50.0 / 56.5
                {22016, 4096, S, 8, 176, true},     // 54.0 / 56.8
                {22016, 4096, S, 8, 208, false},    // 68.0 / 58.3
                {32000, 4096, P, 1, 160, true},     // 66.3 / 81.5
                {32000, 4096, P, 1, 192, true},     // 78.5 / 85.6
                {32000, 4096, P, 1, 224, false},    // 98.7 / 83.4
                {12288, 4096, P, 8, 224, false},    // 47.2 / 38.0
                {4096, 4096, P, 8, 176, false},     // 17.2 / 15.7
                // d 5120, ffn 13824
                {15360, 5120, P, 8, 160, true},     // 46.6 / 52.7
                {15360, 5120, P, 8, 176, true},     // 51.1 / 54.0
                {5120, 5120, P, 8, 160, true},      // 20.7 / 22.8
                {27648, 5120, S, 8, 192, true},     // 83.3 / 94.3
                {5120, 13824, P, 8, 160, true},     // 45.3 / 47.7
                {5120, 13824, P, 8, 176, false},    // 51.1 / 48.2
                {15360, 5120, P, 8, 224, false},    // 61.2 / 54.9
                // d 3072, ffn 8192
                {9216, 3072, P, 8, 160, true},      // 22.8 / 24.5
                {16384, 3072, S, 8, 160, true},     // 31.2 / 33.8
                {9216, 3072, P, 8, 192, false},     // 26.8 / 25.0
                // d 2048, ffn 5504; d 1024, ffn 2752; d 8192, ffn 16384
                {11008, 2048, S, 8, 176, false},    // 23.4 / 20.1
                {6144, 2048, P, 8, 176, false},     // 15.1 / 13.7
                {5504, 1024, S, 8, 160, false},     // 13.1 / 11.3
                {32768, 8192, S, 8, 192, true},     // 139 / 157
            };
            for (const Point& q : points) {
                const ss::GemmPlan p = ss::gemm_plan(q.N, q.Kp, q.rows, q.epi, 256, q.max_ksplit);
                if ((p.sweep_gn > 0) == q.sweep && (p.block >= 0) != q.sweep) continue;
                std::printf("N %d Kp %d, %d rows: the other kernel is chosen\n", q.N, q.Kp, q.rows);
                return 1;
            }
            return 0;
        }
    """)


def test_tile_choice_follows_the_measurements(tmp_path):
    """Block kernel: projections of prompt forwards of which the tile and slices named were measured 9 % or more slower (microseconds with what
    follows) than the ones that are taken."""
    _run(tmp_path, r"""
        struct Point { int N, Kp, epi, rows, tile, ksplit; };
        int main() {
            const int G = ss::EPI_SWIGLU;
            const Point slower[] = {
                {27648, 5120, G, 494, 2, 1},                  // 137.8, with 256 x 256 115.0
                {32768, 6144, G, 494, 2, 1},                  // 170.7 / 150.8
                {28672, 4096, G, 494, 2, 1},                  // 110.4 / 96.0
                {1536, 1536, ss::EPI_RESIDUAL, 2033, 5, 2},   // 32.1, with 128 x 128 26.0
                {6144, 768, G, 2033, 5, 1},                   // 26.8, with 128 x 192 21.2
                {5632, 1024, G, 640, 5, 1},                   // 13.7, with 128 x 128 11.3
                {3072, 1024, ss::EPI_QKV, 272, 6, 2},         // 13.6 with the rotation, whole in 128 x 64 10.4
            };
            for (const Point& q : slower) {
                const ss::GemmPlan p = ss::gemm_plan(q.N, q.Kp, q.rows, q.epi, 256);
                if (p.block != q.tile || p.ksplit != q.ksplit) continue;
                std::printf("N %d Kp %d, %d rows: tile %d\n", q.N, q.Kp, q.rows, q.tile);
                return 1;
            }
            return 0;
        }
    """)
