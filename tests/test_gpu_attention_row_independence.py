"""A row's numbers do not depend on when the other rows of its micro-batch leave: within one 16-row strip the same launches
run, whatever is still alive.  Bit for bit: the sums are the same sums in the same order."""
import numpy as np
import pytest

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu


# 16 heads: 16 rows are 256 (row, head) pairs, 3 rows 48; 32 heads: 512 and 96.  40 and 48 heads: 640 and
# 768, so 4 waves take 8 slices (2 up to 640 pairs at long contexts), and 8 waves as soon as 512 are left.  Contexts on both sides of what 8 waves have
# in flight (256 slots of 128 elements, 512 of 64).
@pytest.mark.parametrize("heads,head_dim,longest", [(16, 64, 600), (16, 64, 505), (32, 128, 300), (32, 128, 250),
                                                    (40, 128, 300), (48, 64, 700), (40, 128, 1100), (36, 64, 2100)])
def test_rows_that_leave_do_not_change_the_others(heads, head_dim, longest):
    shape = synth.ModelShape("leave", 1, heads * head_dim, heads, head_dim, 256, 272)
    gw = ss.Weights(shape, synth.make_weights(shape, seed=8, std=0.04, threads=4))
    rng = np.random.default_rng(longest)
    rows, steps, stay = 16, 10, (0, 7, 15)
    plens = rng.integers(3, 30, rows)
    plens[0] = longest
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]

    def call(cut):
        s = [q if i in stay else q[:len(q) - cut] for i, q in enumerate(seqs)]
        offs = np.concatenate([[0], np.cumsum([len(q) for q in s])]).astype(np.int32)
        out = ss.ss_forward_logits(gw, np.concatenate(s), offs, plens.astype(np.int32))
        at = np.concatenate([[0], np.cumsum([len(q) - p + 1 for q, p in zip(s, plens)])])
        return [out[at[i]:at[i + 1]] for i in stay]

    try:
        all_stay = call(0)
        for cut in (9, 4):
            for i, a, b in zip(stay, all_stay, call(cut)):
                assert np.array_equal(a, b), (cut, i, np.abs(a - b).max())
    finally:
        gw.close()


# The loads beyond a context are skipped from 257 to 1024 (row, head) pairs and issued otherwise.  One row that leaves takes the others over
# that line: 13 to 12 rows of 20 heads, and back over the upper one, 26 to 25 rows of 40.  Contexts at the edges of a load and of a trip.
@pytest.mark.parametrize("heads,head_dim,rows,contexts", [(20, 128, 13, (34, 122, 187, 252, 316, 380, 442, 506, 570, 634)),
                                                          (20, 128, 13, (28, 60, 92, 124, 250, 379, 508, 636, 700, 764)),
                                                          (20, 64, 13, (60, 124, 252, 380, 506, 636, 764, 892, 1020, 1290)),
                                                          (40, 64, 26, (28, 60, 92, 124, 252, 380, 508, 636, 764, 780))])
def test_loads_that_are_skipped_do_not_change_the_sums(heads, head_dim, rows, contexts):
    shape = synth.ModelShape("skip", 1, heads * head_dim, heads, head_dim, 256, 272)
    gw = ss.Weights(shape, synth.make_weights(shape, seed=8, std=0.04, threads=4))
    rng = np.random.default_rng(contexts[-1])
    steps = 8
    plens = np.resize(np.array(contexts), rows)
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]

    def call(cut):   # the last row ends `cut` steps early
        s = seqs[:-1] + [seqs[-1][:len(seqs[-1]) - cut]]
        offs = np.concatenate([[0], np.cumsum([len(q) for q in s])]).astype(np.int32)
        return ss.ss_forward_logits(gw, np.concatenate(s), offs, plens.astype(np.int32))[:(rows - 1) * (steps + 1)]

    try:
        assert np.array_equal(call(0), call(steps))
    finally:
        gw.close()
