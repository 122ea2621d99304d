"""ss_forward_logits hands its logits out in pinned pieces while the next forward runs: outputs of several pieces (more than
the ring holds, copied by host threads), and rows that leave at different steps, arrive whole and in place.  Each sequence
is compared with a call of its own: other launch shapes round an activation to the neighbouring half here and there, which
moves a logit by up to about 1e-3 of the largest; a row in another's place is off by the size of a logit."""
import numpy as np
import pytest

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.mark.parametrize("rows,lens,all_prompt", [(60, 80, True), (9, 200, False), (600, 6, False), (1, 3, False)])
def test_logits_arrive_whole_and_in_place(rows, lens, all_prompt):
    shape = synth.ModelShape("transfer", 1, 256, 4, 64, 256, 2064)
    rng = np.random.default_rng(rows)
    gw = ss.Weights(shape, synth.make_weights(shape, seed=4, threads=1))
    n = rng.integers(max(1, lens // 2), lens + 1, rows).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    toks = rng.integers(0, shape.vocab, int(offs[-1])).astype(np.int32)
    npr = n if all_prompt else rng.integers(1, n + 1).astype(np.int32)
    out = ss.ss_forward_logits(gw, toks, offs, npr, all_prompt_logits=all_prompt)
    at = 0
    for i in range(rows):
        k = int(n[i]) if all_prompt else int(n[i] - npr[i] + 1)
        if i in (0, 1, rows // 3, rows - 1):
            one = ss.ss_forward_logits(gw, toks[offs[i]:offs[i + 1]], [0, int(n[i])], [int(npr[i])], all_prompt_logits=all_prompt)
            assert np.abs(out[at:at + k] - one).max() <= TOL * np.abs(one).max(), i
        at += k
    assert at == len(out)
    gw.close()


def test_steps_of_more_pieces_than_the_ring_holds():
    """163 rows of 32000 logits are six pieces of 4 MiB per forward, the ring holds four: while a step's last pieces wait for
    the copier, the next forward already fills the other buffer, and the one after waits for this one's to have left."""
    shape = synth.ModelShape("ring", 1, 256, 4, 64, 256, 32000)
    rng = np.random.default_rng(3)
    gw = ss.Weights(shape, synth.make_weights(shape, seed=4, threads=8))
    rows, steps = 163, 5
    plens = rng.integers(1, 9, rows).astype(np.int32)
    n = (plens + rng.integers(steps - 1, steps + 1, rows)).astype(np.int32)   # some rows leave one step early
    offs = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    toks = rng.integers(0, shape.vocab, int(offs[-1])).astype(np.int32)
    out = ss.ss_forward_logits(gw, toks, offs, plens)
    at = np.concatenate([[0], np.cumsum(n - plens + 1)])
    assert at[-1] == len(out)
    for i in range(0, rows, 9):
        one = ss.ss_forward_logits(gw, toks[offs[i]:offs[i + 1]], [0, int(n[i])], [int(plens[i])])
        assert np.abs(out[at[i]:at[i + 1]] - one).max() <= TOL * np.abs(one).max(), i
    for _ in range(3):
        assert np.array_equal(ss.ss_forward_logits(gw, toks, offs, plens), out)
    gw.close()
