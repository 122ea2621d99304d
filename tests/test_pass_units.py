"""How a group pass hands its micro-batches out: host arithmetic, compiled and run on the CPU."""
from test_projection_plans import _run, pytestmark  # noqa: F401


def test_every_lane_has_work_while_there_is_some(tmp_path):
    """Every micro-batch is handed out once, in order; only several together share, and beside each such unit run as many lanes as
    the units that are left leave free, however few of the micro-batches can share."""
    _run(tmp_path, r"""
        #include <algorithm>
        #include <cstdlib>
        int main() {
            std::srand(6);
            int filled = 0;
            for (int t = 0; t < 200000; ++t) {
                const int n = 1 + std::rand() % 12, lanes = std::min(n, 1 + std::rand() % 4);
                std::vector<int> order(n), rows(n), seen(n, 0), at(n);
                std::vector<char> can(n);
                const int odds = std::rand() % 4;
                for (int k = 0; k < n; ++k) {
                    order[k] = k;
                    rows[k] = 1 + std::rand() % ss::kSharedMbRows;
                    can[k] = lanes > 1 && (odds == 0 || std::rand() % 4 < odds);
                }
                for (int k = n; k-- > 1;) std::swap(order[k], order[std::rand() % (k + 1)]);
                for (int i = 0; i < n; ++i) at[order[i]] = i;
                const ss::PassUnits p = ss::pass_units(order, rows, can, lanes);
                if (p.beside.size() != p.shared.size()) return 1;
                int last = -1;
                for (const auto& u : p.alone) {
                    if (u.size() != 1 || at[u[0]] < last) return 2;
                    last = at[u[0]];
                    ++seen[u[0]];
                }
                last = -1;
                int most_after = 0, alone_that_can = 0;
                for (size_t u = p.shared.size(); u-- > 0;) {
                    most_after = std::max(most_after, (int)p.shared[u].size());
                    if (p.shared[u].size() < 2 || p.beside[u] + most_after != lanes) {
                        std::printf("%d lanes, a unit of %d: %d beside\n", lanes, (int)p.shared[u].size(), p.beside[u]);
                        return 3;
                    }
                }
                for (const auto& u : p.shared) {
                    int r = 0;
                    for (int k : u) {
                        if (!can[k] || at[k] < last) return 4;
                        last = at[k];
                        ++seen[k];
                        r += rows[k];
                    }
                    if (r > ss::kSharedRows) return 5;
                }
                for (const auto& u : p.alone) alone_that_can += can[u[0]];
                if (alone_that_can > 1) return 6;   // the left-over
                for (int k = 0; k < n; ++k)
                    if (seen[k] != 1) return 7;
                filled += !p.shared.empty() && !p.alone.empty();
            }
            return filled ? 0 : 8;
        }
    """)
