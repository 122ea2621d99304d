"""Prompt forwards whose unsliced projections finish their results themselves (rotation, key/value slots, residual stream)
and those that leave it to the next launch, on both head sizes and widths that end inside a tile, each followed by decode
steps on the slots they wrote; against the oracle."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": synth.ModelShape("epi64", 2, 320, 5, 64, 720, 528),
    "hd128": synth.ModelShape("epi128", 2, 640, 5, 128, 1328, 528),
    "deep": synth.ModelShape("epideep", 2, 1536, 12, 128, 1024, 528),   # k long enough for slices below 2048 token-rows
}
# six roundings of projection inputs to 11 bits per layer and the slots' two, two layers: 2^-11 * sqrt(16) ~ 2e-3 of the
# residual stream, and the worst of some thousand logits 3 to 4 standard deviations of a tenth of that
TOL = 3e-3


@pytest.fixture(scope="module", params=sorted(SHAPES))
def model(request, oracle_built):
    shape = SHAPES[request.param]
    W = synth.make_weights(shape, seed=21, norm_jitter=0.1, threads=1)
    gw = ss.Weights(shape, W)
    yield shape, gw, OracleModel(shape, W, "f32")
    gw.close()


@pytest.mark.parametrize("rows", [145, 255, 272, 531, 1100])
def test_prompt_then_decode_match_the_oracle(model, rows):
    shape, gw, om = model
    rng = np.random.default_rng(rows)
    plens, left = [], rows
    while left > 0:
        plens.append(int(min(left, rng.integers(1, 130))))
        left -= plens[-1]
    steps = 2
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    offs = np.concatenate([[0], np.cumsum([len(q) for q in seqs])]).astype(np.int32)
    got = ss.ss_forward_logits(gw, np.concatenate(seqs), offs, np.array(plens, np.int32))
    assert np.isfinite(got).all()
    for i in sorted({0, len(plens) // 2, len(plens) - 1, int(np.argmax(plens)), int(np.argmin(plens))}):
        ref = om.teacher_forced(seqs[i], first=plens[i] - 1)
        mine = got[i * (steps + 1):(i + 1) * (steps + 1)]
        err = np.abs(mine - ref).max() / np.abs(ref).max()
        assert err <= TOL, (rows, i, plens[i], err)
