"""The plans of the kernel for decode forwards of few rows (host arithmetic, compiled and run on the CPU): every k-block of every
unit belongs to exactly one wave's chain, a workgroup has no more waves, LDS and pieces to copy than the kernel is built for."""
from test_projection_plans import _run, pytestmark  # noqa: F401


def test_every_group_of_a_unit_is_summed_once(tmp_path):
    _run(tmp_path, r"""
        #include <algorithm>
        #include <vector>
        int main() {
            int plans = 0;
            const int rc = every_matrix([&](const Mat& m) {
                for (int cu : {64, 256, 304})
                    for (int n = 1; n <= 5; ++n)
                        for (int res = 0; res < (m.epi == ss::EPI_PARTIAL ? 2 : 1); ++res) {
                            const int epi = res ? ss::EPI_RESIDUAL : m.epi;
                            const ss::FewPlan p = ss::few_plan(m.N, m.Kp, n, epi, cu, m.max_ksplit);
                            if (!p.units_wg) continue;
                            ++plans;
                            const ss::GemmPlan g = ss::gemm_plan(m.N, m.Kp, n, m.epi, cu, m.max_ksplit);
                            const int KB = m.Kp / 32;
                            bool ok = n <= ss::kFewRows && g.narrow && g.block < 0 && m.Kp % 128 == 0 && p.kb_slice % 4 == 0 && p.items == g.ksplit * p.parts;
                            ok = ok && p.items * p.units_wg <= ss::kFewWaves && ss::few_lds_bytes(n, m.Kp, epi) <= 160 * 1024;
                            ok = ok && (m.Kp / 8) * n <= 4 * n * 64 * ss::kFewWaves && m.N % (m.epi == ss::EPI_SWIGLU ? 32 : 16) == 0;
                            std::vector<int> seen(KB / 4);
                            for (int item = 0; ok && item < p.items; ++item) {   // as the kernel deals them out
                                const int slice = item / p.parts, part = item % p.parts;
                                const int s0 = slice * p.kb_slice, s1 = std::min(KB, s0 + p.kb_slice), G = std::max(s1 - s0, 0) / 4;
                                int first = s0 / 4, step = 1, count = G;
                                if (p.wave_kb && p.parts == 4) {
                                    const int quarter = ((std::max(s1 - s0, 0) + 3) / 4 + 3) / 4;
                                    first += std::min(G, part * quarter);
                                    count = std::min(G, (part + 1) * quarter) - std::min(G, part * quarter);
                                } else if (p.parts == 2) {
                                    first += part;
                                    step = 2;
                                    count = (G - part + 1) / 2;
                                }
                                for (int i = 0; i < count; ++i) {
                                    const int at = first + i * step;
                                    ok = ok && at >= 0 && at < KB / 4;
                                    if (ok) ++seen[at];
                                }
                            }
                            for (int c : seen) ok = ok && c == 1;
                            if (ok) continue;
                            std::printf("N %d Kp %d epilogue %d rows %d cu %d: items %d parts %d units %d\n", m.N, m.Kp, epi, n, cu, p.items, p.parts, p.units_wg);
                            return 1;
                        }
                return 0;
            });
            return rc ? rc : plans > 100 ? 0 : 2;
        }
    """)
