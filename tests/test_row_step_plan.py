"""When a decode step goes through k_row_step: host arithmetic, compiled and run on the CPU."""
from test_projection_plans import _run, pytestmark  # noqa: F401


def test_row_step_plan_keeps_to_what_the_kernel_can_do(tmp_path):
    _run(tmp_path, r"""
        int main() {
            int taken = 0;
            for (int cu : {64, 256, 304})
                for (int L : {1, 2, 16, 17})
                    for (int d = 64; d <= 1024; d += 64)
                        for (int F : {16, 176, 688, 8192, 8208})
                            for (int V : {16, 1024, 32000})
                                for (int n : {1, 16, 17, 64, 256, 257, 304, 305})
                                    for (int ctx : {1, 300, 4096}) {
                                        const bool yes = ss::row_step_plan(L, d, F, V, n, ctx, cu);
                                        taken += yes;
                                        // whole strips: a shrinking micro-batch keeps its route inside one
                                        if (yes != ss::row_step_plan(L, d, F, V, (n + 15) / 16 * 16, ctx, cu)) return 1;
                                        // fewer slots never take it off the route
                                        if (yes && !ss::row_step_plan(L, d, F, V, n, (ctx + 1) / 2, cu)) return 2;
                                        if (!yes) continue;
                                        if (n > cu || L > ss::kRowMaxLayers || d > 64 * ss::kRowWaves || F > ss::kRowMaxFfn) return 3;
                                        for (int hd : {64, 128})   // a wave per head, and LDS within what every launch may have
                                            if (d / hd > ss::kRowWaves || ss::row_step_lds_bytes(d, (F + 63) / 64 * 64, hd) > (64u << 10))
                                                return 4;
                                    }
            if (!taken || ss::row_step_plan(32, 4096, 11008, 32000, 1, 1, 256)) return 5;
            for (int mode : {1, 2, 4, 8, 16, 80}) {   // the testing aids keep the projection kernels
                ss::set_gemm_mode(mode);
                if (ss::row_step_plan(2, 256, 688, 1024, 16, 40, 256)) return 6;
            }
            ss::set_gemm_mode(0);
            return ss::row_step_plan(2, 256, 688, 1024, 16, 40, 256) ? 0 : 7;
        }
    """)
