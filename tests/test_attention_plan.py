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
                    shares = shares && !ss::attention_may_widen(rows[k], H, mb[k].prompt + cap, hd) &&
                             ss::attention_wide(ss::kSharedMbRows, rows[k], H) == ss::attention_wide(ss::kSharedMbRows, rows[0], H);
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
