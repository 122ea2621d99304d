"""Launch shapes of the decode attention: host arithmetic, compiled and run on the CPU."""
from test_projection_plans import _run, pytestmark  # noqa: F401


def test_shares_fit_the_smallest_workspace(tmp_path):
    """The workgroups that share out a row's slots leave their sums in an activation buffer, which holds kWorkspaceRows rows of the
    model's width and no more where prompts are short: every head count and size that the library takes, every row count and
    contexts around every whole number of shares."""
    _run(tmp_path, r"""
        int main() {
            int split = 0;
            for (int hd : {64, 128})
                for (int H = 1; H * hd <= 8192; ++H)
                    for (int rows = 1; rows <= 130; ++rows)
                        for (int ctx = 255; ctx <= 4097; ctx += (ctx & 1) ? 1 : 127) {
                            const int S = ss::attention_split(rows, H, hd, ctx);
                            if (S < 1 || S > ss::kAttnMaxSplit) return 1;
                            if (S == 1) continue;
                            ++split;
                            if (ss::attention_share_floats(rows, H, hd, S) > (size_t)ss::kWorkspaceRows * H * hd) {
                                std::printf("%d heads of %d, %d rows, context %d: %d shares\n", H, hd, rows, ctx, S);
                                return 2;
                            }
                            if (ctx / S < ss::kAttnSplitSlots) return 3;
                        }
            return split ? 0 : 4;
        }
    """)


def test_slots_are_shared_out_where_that_was_measured_faster(tmp_path):
    """Split or 16 waves a pair, wherever one of them was measured 1.5 % faster or more (a decode step's time per layer)."""
    _run(tmp_path, r"""
        struct Point { int rows, H, hd, ctx; bool split; };
        int main() {
            const Point points[] = {
                // us, 16 waves / split
                {1, 32, 128, 1030, true},    // 57.0 / 56.2
                {3, 32, 128, 1300, true},    // 68.1 / 66.0
                {4, 32, 128, 2000, false},   // 104 / 106
                {6, 16, 128, 1300, true},    // 51.9 / 49.7
                {12, 8, 128, 1300, true},    // 46.9 / 44.8
                {16, 4, 128, 1030, true},    // 39.7 / 38.0
                {24, 4, 128, 1300, true},    // 46.7 / 44.4
                {1, 32, 64, 1030, false},    // 38.1 / 38.8
                {3, 32, 64, 1030, false},    // 39.5 / 41.4
                {6, 16, 64, 1030, false},    // 34.7 / 36.7
                {12, 8, 64, 1030, false},    // 35.0 / 36.0
                {12, 4, 64, 1030, false},    // 29.3 / 29.9
                {24, 4, 64, 1030, false},    // 34.7 / 35.3
                {2, 16, 64, 1300, true},     // 35.4 / 34.5
                {6, 8, 64, 1300, true},      // 35.3 / 34.3
                {12, 4, 64, 1300, true},     // 33.2 / 32.1
                {1, 32, 64, 1600, true},     // 39.7 / 39.0
                {3, 32, 64, 2100, true},     // 49.4 / 47.2
                {4, 16, 64, 2100, true},     // 42.1 / 39.1
                {12, 8, 64, 2100, true},     // 41.8 / 39.8
            };
            for (const Point& q : points) {
                if ((ss::attention_plan(q.rows, q.rows, q.rows, q.H, q.hd, q.ctx).split > 1) == q.split) continue;
                std::printf("%d rows, %d heads of %d, context %d\n", q.rows, q.H, q.hd, q.ctx);
                return 1;
            }
            return 0;
        }
    """)


def test_waves_follow_the_measurements(tmp_path):
    """The waves of a pair, wherever one count was measured 1.5 % faster than the next or more (a decode step's time per layer)."""
    _run(tmp_path, r"""
        struct Point { int rows, H, hd, ctx, waves; };
        int main() {
            const Point points[] = {
                // us, 8 waves / 4
                {8, 32, 128, 900, 8},     // 76.2 / 79.5
                {8, 32, 128, 3000, 8},    // 128.8 / 137.3
                {9, 32, 128, 1200, 4},    // 99.4 / 96.5
                {9, 32, 128, 3000, 4},    // 155.3 / 143.0
                {11, 32, 128, 700, 4},    // 80.6 / 79.2
                {12, 32, 128, 900, 4},    // 92.3 / 89.9
                {12, 32, 128, 1500, 4},   // 112.8 / 110.3
                {16, 16, 128, 1500, 8},   // 72.0 / 77.9
                {20, 16, 128, 1500, 4},   // 92.0 / 87.5
                {24, 16, 128, 900, 4},    // 75.8 / 73.8
                {8, 32, 64, 1500, 8},     // 55.1 / 60.1
                {10, 32, 64, 900, 8},     // 52.6 / 54.3
                {11, 32, 64, 300, 8},     // 41.8 / 42.8
                {12, 32, 64, 1500, 4},    // 65.0 / 63.4
                {11, 32, 64, 3000, 4},    // 89.4 / 85.0
                {18, 16, 64, 900, 8},     // 45.4 / 47.7
                {20, 16, 64, 1500, 4},    // 60.5 / 58.7
                {16, 32, 64, 500, 8},     // 46.8 / 48.0
                // 4 waves / 2
                {17, 32, 128, 400, 4},    // 83.6 / 85.6
                {17, 32, 128, 1500, 2},   // 149.8 / 147.7
                {18, 32, 128, 3000, 2},   // 235.9 / 227.5
                {13, 40, 128, 2200, 2},   // 192.5 / 186.4
                {33, 16, 128, 1500, 2},   // 127.9 / 124.3
                {9, 64, 128, 3000, 2},    // 287.8 / 278.4
                {17, 32, 64, 1000, 4},    // 68.7 / 71.1
                {33, 16, 64, 1000, 4},    // 65.3 / 67.7
                {17, 32, 64, 3000, 2},    // 123.8 / 122.0
            };
            for (const Point& q : points) {
                const ss::AttentionPlan p = ss::attention_plan(q.rows, q.rows, q.rows, q.H, q.hd, q.ctx);
                if (p.waves == q.waves) continue;
                std::printf("%d rows, %d heads of %d, context %d: %d waves\n", q.rows, q.H, q.hd, q.ctx, p.waves);
                return 1;
            }
            return 0;
        }
    """)


def test_shared_forwards_keep_every_member_s_sums(tmp_path):
    """In every forward of micro-batches that share theirs, the attention's slices and shares are those that each of them gets alone:
    also when the one with the longest prompt has ended and those that remain run on."""
    _run(tmp_path, r"""
        #include <cstdlib>
        int main() {
            std::srand(5);
            int checked = 0;
            for (int t = 0; t < 20000; ++t) {
                const int hd = t & 1 ? 64 : 128, H = 1 + std::rand() % (8192 / hd), n = 2 + std::rand() % 3;
                ss::SharedShape mb[4];
                int rows[4], all = 0, most = 0, last = 0;
                bool shares = true;
                for (int k = 0; k < n; ++k) {
                    rows[k] = 1 + std::rand() % (std::rand() % 2 ? 4 : ss::kSharedMbRows);
                    mb[k] = {1 + std::rand() % (std::rand() % 2 ? 60 : 1200), 0};
                    const int cap = 1 + std::rand() % (std::rand() % 2 ? 60 : 700);
                    mb[k].steps = 1 + std::rand() % cap;
                    shares = shares && !ss::attention_may_widen(rows[k], H, mb[k].prompt + cap, hd);
                    all += rows[k];
                    most = rows[k] > most ? rows[k] : most;
                    last = mb[k].steps > last ? mb[k].steps : last;
                }
                if (!shares) continue;
                for (int g = 1; g < last; ++g)
                    for (int live : {all, 1})
                        for (int k = 0; k < n; ++k) {
                            if (mb[k].steps <= g) continue;
                            const ss::AttentionPlan a = ss::attention_plan(live, ss::kSharedMbRows, most, H, hd, ss::shared_context(mb, n, g));
                            const ss::AttentionPlan b = ss::attention_plan(rows[k], rows[k], rows[k], H, hd, mb[k].prompt + g);
                            ++checked;
                            if (a.slices == b.slices && a.split == b.split) continue;
                            std::printf("%d heads of %d, forward %d, %d rows from prompt %d: %d slices, alone %d\n", H, hd, g, rows[k],
                                        mb[k].prompt, a.slices, b.slices);
                            return 1;
                        }
            }
            return checked > 100000 ? 0 : 2;
        }
    """)


def test_a_shrinking_micro_batch_keeps_its_slices_and_gains_waves(tmp_path):
    """Inside a strip the slices (the order of the sums) stay the same for every count of live rows; 8 waves take a pair's slots
    as soon as at most 256 pairs are alive, or 512 in short contexts."""
    _run(tmp_path, r"""
        int main() {
            int fewer = 0;
            for (int hd : {64, 128})
                for (int H = 1; H * hd <= 8192; ++H)
                    for (int mb = 1; mb <= 300; ++mb)
                        for (int ctx : {40, 300, 700, 2001}) {
                            ss::AttentionPlan strip{};
                            for (int n = mb; n >= 1; --n) {
                                const ss::AttentionPlan p = ss::attention_plan(n, n, mb, H, hd, ctx);
                                if (n < mb && n % 16 && (p.slices != strip.slices || p.split != strip.split)) {
                                    std::printf("%d heads of %d, %d of %d rows, context %d: %d slices, %d\n", H, hd, n, mb, ctx, p.slices, strip.slices);
                                    return 1;
                                }
                                strip = p;
                                if (p.waves < (n * H <= (ctx < 600 ? 512 : 256) ? 8 : n * H <= 512 || ctx < 1000 ? 4 : 2) || p.slices < p.waves || p.slices % p.waves) {
                                    std::printf("%d heads of %d, %d of %d rows, context %d: %d waves, %d slices\n", H, hd, n, mb, ctx, p.waves, p.slices);
                                    return 2;
                                }
                                fewer += p.waves < p.slices;
                            }
                        }
            return fewer ? 0 : 3;
        }
    """)
