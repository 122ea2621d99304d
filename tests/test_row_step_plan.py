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


def test_row_step_is_taken_where_it_was_measured_faster(tmp_path):
    """Launches or k_row_step, wherever one of them was measured clearly faster."""
    _run(tmp_path, r"""
        struct Point { int L, d, hd, F, V, rows, ctx; bool row; };
        int main() {
            const Point points[] = {
                // us, launches / row step
                {2, 256, 64, 688, 1024, 16, 20, true},      // 63.0 / 48.1
                {2, 256, 64, 688, 1024, 1, 200, true},      // 62.3 / 54.0
                {2, 256, 64, 688, 1024, 16, 1000, false},   // 76.8 / 80.9
                {2, 256, 64, 688, 1024, 100, 600, true},    // 115 / 70
                {1, 64, 64, 176, 16000, 1, 8, false},       // 36.1 / 77.4
                {1, 64, 64, 176, 16000, 16, 500, false},    // 40.9 / 79.7
                {1, 64, 64, 176, 6000, 1, 8, false},        // 35.0 / 40.5
                {1, 64, 64, 176, 6000, 100, 200, true},     // 51.7 / 43.2
                {1, 64, 64, 176, 2000, 1, 8, true},         // 34.2 / 25.7
                {1, 64, 64, 4096, 1008, 1, 8, false},       // 36.9 / 62.6
                {4, 64, 64, 2048, 1008, 16, 200, false},    // 111 / 131
                {4, 128, 128, 2048, 1024, 1, 8, false},     // 105 / 136
                {4, 128, 128, 2048, 1024, 100, 8, true},    // 156 / 136
                {2, 128, 64, 352, 8000, 1, 200, false},     // 61.2 / 65.2
                {2, 192, 64, 512, 4096, 1, 8, true},        // 58.4 / 52.9
                {2, 192, 64, 512, 4096, 1, 600, false},     // 64.2 / 71.0
                {2, 320, 64, 320, 512, 1, 200, false},      // 60.8 / 66.0
                {2, 320, 64, 320, 512, 100, 200, true},     // 104 / 71
                {16, 64, 64, 176, 32000, 16, 8, true},      // 362 / 276
            };
            for (const Point& q : points) {
                if (ss::row_step_plan(q.L, q.d, q.F, q.V, q.rows, q.ctx, 256, q.hd) == q.row) continue;
                std::printf("%d layers %d wide, ffn %d, %d ids, %d rows, context %d\n", q.L, q.d, q.F, q.V, q.rows, q.ctx);
                return 1;
            }
            // more rows never take a micro-batch off the route while there are units for them
            for (int L : {1, 2, 16})
                for (int d = 64; d <= 512; d += 64)
                    for (int F : {16, 688, 4096})
                        for (int V : {16, 1024, 16000})
                            for (int ctx : {8, 300, 4000})
                                for (int n = 16; n < 256; n += 16)
                                    if (ss::row_step_plan(L, d, F, V, n, ctx, 256) && !ss::row_step_plan(L, d, F, V, n + 16, ctx, 256)) return 2;
            return 0;
        }
    """)
