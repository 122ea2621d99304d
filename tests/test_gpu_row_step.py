"""The decode step of a small model in one workgroup per row (k_row_step): heads that do not divide the waves, odd last
strips, inner sizes that end inside a group of k-blocks, fewer strips than waves, contexts around what a wave has in flight
(HD 64: 32 slots a wave, HD 128: 16); against the oracle, and against the launches that it replaces."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [
    synth.ModelShape("hd64x3", 2, 192, 3, 64, 176, 272),     # 2 waves a head and 2 idle; 17 strips of head
    synth.ModelShape("hd64x8", 1, 512, 8, 64, 80, 1040),     # a wave a head; 65 strips
    synth.ModelShape("hd64x1", 3, 64, 1, 64, 16, 16),        # everything smaller than the waves; one strip of head
    synth.ModelShape("hd128x1", 2, 128, 1, 128, 688, 512),   # 8 waves for the only head
    synth.ModelShape("hd128x4", 1, 512, 4, 128, 400, 256),
]
# Six projection inputs, keys and values per layer, each rounded to 11 bits (2^-12 at worst, a third of that on average), up
# to three layers: 5 * 2^-12 / sqrt(3) = 7e-4 of the logits' size in the mean, 4 times that at most.
TOL = 3e-3


def _offs(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


@pytest.fixture(scope="module", params=SHAPES, ids=lambda s: s.name)
def model(request, oracle_built):
    W = synth.make_weights(request.param, seed=21, std=0.05, norm_jitter=0.1, threads=1)
    gw = ss.Weights(request.param, W)
    yield request.param, gw, OracleModel(request.param, W, "f64")
    gw.close()


@pytest.mark.parametrize("rows,longest", [(1, 130), (9, 33), (17, 65), (40, 257)])
def test_logits(model, rows, longest):
    shape, gw, om = model
    rng = np.random.default_rng(rows)
    plens = rng.integers(1, 20, rows)
    plens[:3] = (longest, longest - 1, longest - 2)[:min(3, rows)]
    steps = 3
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    args = (gw, np.concatenate(seqs), _offs([len(q) for q in seqs]), plens.astype(np.int32))
    got = ss.ss_forward_logits(*args)
    ss.ss_set_gemm_mode(1)   # projection kernels one by one
    try:
        launches = ss.ss_forward_logits(*args)
    finally:
        ss.ss_set_gemm_mode(0)
    assert np.abs(got - launches).max() <= TOL * np.abs(launches).max()
    for i in sorted({0, 1 % rows, 2 % rows, rows - 1}):
        ref = om.teacher_forced(seqs[i], first=int(plens[i]) - 1)
        err = np.abs(got[i * (steps + 1):(i + 1) * (steps + 1)] - ref).max() / np.abs(ref).max()
        assert err <= TOL, (shape.name, rows, i, err)


@pytest.mark.parametrize("flags", [0, ss.SS_COMPACT])
def test_tokens_are_the_argmax_of_the_logits(model, flags):
    """Greedy tokens (known ends: all steps of a row in one launch) against the argmax of the logits of the same forwards,
    one launch each; a row's numbers do not depend on the others.  Slots written by one step are read by the next, across what
    a wave has in flight."""
    shape, gw, _ = model
    rng = np.random.default_rng(7)
    plens = rng.integers(2, 30, 12)
    plens[:2] = (100, 1)
    targets = rng.integers(1, 40, 12).astype(np.int32)
    prompts = [rng.integers(0, shape.vocab, p).astype(np.int32) for p in plens]
    r = ss.ss_decode_microbatch(gw, np.concatenate(prompts), _offs(plens), 40, targets, flags)
    assert np.array_equal(r["lens"], targets)
    assert all((r["tokens"][i, t:] == -1).all() for i, t in enumerate(targets))
    seqs = [np.concatenate([p, r["tokens"][i, :targets[i] - 1]]) for i, p in enumerate(prompts)]
    lg = ss.ss_forward_logits(gw, np.concatenate(seqs), _offs([len(q) for q in seqs]), plens.astype(np.int32))
    at = 0
    for i, t in enumerate(targets):
        assert np.array_equal(lg[at:at + t].argmax(-1), r["tokens"][i, :t]), i
        at += t
