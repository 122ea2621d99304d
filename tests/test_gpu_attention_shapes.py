"""Attention at the edges of its tiles, both head sizes, against the oracle: prompts around 16, 64, 128 and 256 slots (one
or two query tiles per wave: the longest row decides), and decode steps whose contexts cross what 16, 8 and 4 waves have in
flight, at row counts on both sides of the choice between them."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": synth.ModelShape("att64", 1, 256, 4, 64, 256, 272),
    "hd128": synth.ModelShape("att128", 1, 512, 4, 128, 256, 272),
}
# One layer.  Projection inputs, slots and probabilities are rounded to 11 bits: 2e-3 of the largest logit where scores are
# small.  Here they have a spread of 3.3 (0.08^2 * 512, per element of q and k), so keys rounded by up to 2^-12 of their
# value move a score by 3.3 * 2^-12 / sqrt(3) = 5e-4 (standard deviation), four of which are another 2e-3 of a probability.
TOL = 4e-3


@pytest.fixture(scope="module", params=sorted(SHAPES))
def model(request, oracle_built):
    shape = SHAPES[request.param]
    # wide matrices: scores of several units, so that the softmax is neither flat nor a single slot
    W = synth.make_weights(shape, seed=33, std=0.08, norm_jitter=0.1, threads=1)
    gw = ss.Weights(shape, W)
    yield shape, gw, OracleModel(shape, W, "f32")
    gw.close()


def _offs(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


@pytest.mark.parametrize("lens", [[1, 15, 16, 17, 40], [31, 63, 64, 65, 2], [127, 128, 129, 80, 255], [256, 1, 64, 33],
                                  [257, 130, 127, 16], [700, 5, 320]], ids=lambda v: "x".join(map(str, v)))
def test_every_position_of_a_prompt(model, lens):
    shape, gw, om = model
    rng = np.random.default_rng(sum(lens))
    offs = _offs(lens)
    toks = rng.integers(0, shape.vocab, offs[-1]).astype(np.int32)
    got = ss.ss_forward_logits(gw, toks, offs, np.array(lens, np.int32), all_prompt_logits=True)
    for i in range(len(lens)):
        ref = om.teacher_forced(toks[offs[i]:offs[i + 1]], first=0)
        err = np.abs(got[offs[i]:offs[i + 1]] - ref).max() / np.abs(ref).max()
        assert err <= TOL, (lens, i, err)


@pytest.mark.parametrize("rows,longest", [(1, 1030), (3, 600), (48, 530), (49, 520), (128, 270), (129, 260)])
def test_decode_steps(model, rows, longest):
    shape, gw, om = model
    rng = np.random.default_rng(rows)
    plens = rng.integers(1, 40, rows)
    plens[0] = longest
    plens[rows // 2] = longest // 2 if rows > 1 else longest
    steps = 3
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    got = ss.ss_forward_logits(gw, np.concatenate(seqs), _offs([len(q) for q in seqs]), plens.astype(np.int32))
    for i in sorted({0, rows // 2, rows - 1}):
        ref = om.teacher_forced(seqs[i], first=int(plens[i]) - 1)
        mine = got[i * (steps + 1):(i + 1) * (steps + 1)]
        err = np.abs(mine - ref).max() / np.abs(ref).max()
        assert err <= TOL, (rows, i, err)
