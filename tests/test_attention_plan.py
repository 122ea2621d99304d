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
