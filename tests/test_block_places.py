"""The order in which the block kernel takes its tiles (host arithmetic, compiled and run on the CPU): every tile is some workgroup's,
and only one's, whether each die keeps row tiles of its own or not and whatever is left over."""
from test_projection_plans import _run, pytestmark  # noqa: F401


def test_every_tile_is_one_workgroups(tmp_path):
    _run(tmp_path, r"""
        #include <algorithm>
        #include <vector>
        int main() {
            std::vector<int> heights;
            for (const ss::BlockTile& t : ss::block_tiles) heights.push_back(t.ms);
            for (int ms : heights)
                for (int n : {1, 2, 3, 7, 8, 11, 16, 21, 27, 86, 115, 250})
                    for (int m = 1; m <= 100; ++m) {
                        std::vector<int> seen(n * m);
                        for (int b = 0; b < n * m; ++b) {
                            const ss::BlockPlace p = ss::block_place(b, n, m, ms);
                            if (p.n_tile >= 0 && p.n_tile < n && p.m_tile >= 0 && p.m_tile < m) ++seen[p.n_tile * m + p.m_tile];
                            // where a die keeps its own row tiles, they are the same ones through all columns
                            const int own = ms >= ss::kBlockOwnStrips && m >= 8 * ss::kBlockOwnFrom ? m / 8 : 0;
                            if (b / 8 < own * n && (p.m_tile / own != b % 8 || p.n_tile != b / 8 / own)) return 2;
                        }
                        for (int s : seen)
                            if (s != 1) {
                                std::printf("tiles of %d strips, %d x %d of them\n", ms, m, n);
                                return 1;
                            }
                    }
            return 0;
        }
    """)
