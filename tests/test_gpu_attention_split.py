"""Decode attention whose slots several workgroups share out (few pairs, long contexts): contexts around its beginning and around
whole shares, short rows beside a long one (shares without a slot), both head sizes, against the oracle; few heads and short
prompts, where the buffer of the shares is smallest; a row's numbers while the others leave; and the other way round, slightly more than two
pairs for each unit, whose slots go to two waves."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": synth.ModelShape("split64", 1, 512, 8, 64, 256, 272),
    "hd128": synth.ModelShape("split128", 1, 512, 4, 128, 256, 272),
}
TOL = 4e-3   # as for decode attention in general: one layer, 11-bit inputs, slots and scores with a spread of some units


@pytest.fixture(scope="module", params=sorted(SHAPES))
def model(request, oracle_built):
    shape = SHAPES[request.param]
    W = synth.make_weights(shape, seed=34, std=0.08, norm_jitter=0.1, threads=1)
    gw = ss.Weights(shape, W)
    ss.ss_set_gemm_mode(1)   # small models would go through k_row_step
    yield shape, gw, OracleModel(shape, W, "f32")
    ss.ss_set_gemm_mode(0)
    gw.close()


def _forced(gw, seqs, plens):
    offs = np.concatenate([[0], np.cumsum([len(q) for q in seqs])]).astype(np.int32)
    return ss.ss_forward_logits(gw, np.concatenate(seqs), offs, np.array(plens, np.int32))


@pytest.mark.parametrize("plens", [[1022], [1087, 3], [1278], [1790, 5, 64, 1000, 1791, 300, 2], [1535, 64, 1, 700], [4000, 2, 255, 256, 257, 1025, 320, 63, 2049, 17, 1, 640]],
                         ids=lambda v: "x".join(map(str, v)))
def test_logits(model, plens):
    shape, gw, om = model
    rng = np.random.default_rng(sum(plens))
    steps = 4
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    got = _forced(gw, seqs, plens)
    for i in range(min(len(plens), 5)):
        ref = om.teacher_forced(seqs[i], first=plens[i] - 1)
        err = np.abs(got[i * (steps + 1):(i + 1) * (steps + 1)] - ref).max() / np.abs(ref).max()
        assert err <= TOL, (plens, i, err)


def test_rows_that_leave_do_not_change_the_others(model):
    shape, gw, _ = model
    rng = np.random.default_rng(3)
    plens, steps = [1300, 40, 900, 1100], 6
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    whole = _forced(gw, seqs, plens)
    cut = _forced(gw, [seqs[0]] + [q[:len(q) - 4] for q in seqs[1:]], plens)
    assert np.array_equal(whole[:steps + 1], cut[:steps + 1])


@pytest.mark.parametrize("pairs", [520, 640])
@pytest.mark.parametrize("longest", [1001, 2003])   # 1000 slots of 128 elements and 2000 of 64 are the lines
def test_two_waves_a_pair(model, pairs, longest):
    shape, gw, om = model
    rows = pairs // shape.n_heads
    rng = np.random.default_rng(rows)
    plens = rng.integers(1, 30, rows)
    plens[[0, rows // 2]] = longest - 2, 700
    steps = 3
    seqs = [rng.integers(0, shape.vocab, p + steps).astype(np.int32) for p in plens]
    got = _forced(gw, seqs, plens)
    for i in (0, 1, rows // 2, rows - 1):
        ref = om.teacher_forced(seqs[i], first=plens[i] - 1)
        err = np.abs(got[i * (steps + 1):(i + 1) * (steps + 1)] - ref).max() / np.abs(ref).max()
        assert err <= TOL, (rows, i, err)


# Prompts of 5 tokens: activation buffers of 128 rows, the smallest there are.  4 heads of 64 and 24 rows, 2 of 128 and 42 rows
# fill the buffer with shares; 1 head of 64 and 90 rows has no room for a second one.
# (In mode 0 the first model's steps leave k_row_step by themselves at about 1350 slots.)
FEW = [(4, 64, 24, 1900, 0), (2, 128, 42, 1300, 1), (1, 64, 90, 1100, 1)]


@pytest.mark.parametrize("heads,hd,rows,steps,mode", FEW, ids=lambda v: str(v))
def test_few_heads_and_short_prompts(oracle_built, heads, hd, rows, steps, mode):
    """Both entry points give the same tokens, the oracle's wherever its two largest logits are apart; the same tokens given as
    inputs have its logits."""
    shape = synth.ModelShape("few", 1, heads * hd, heads, hd, 256, 272)
    W = synth.make_weights(shape, seed=35, std=0.08, norm_jitter=0.1, threads=1)
    om = OracleModel(shape, W, "f32")
    gw = ss.Weights(shape, W)
    rng = np.random.default_rng(heads)
    plen = 5
    toks = rng.integers(0, shape.vocab, rows * plen).astype(np.int32)
    offs = (np.arange(rows + 1) * plen).astype(np.int32)
    limits = np.full(rows, steps, np.int32)
    ss.ss_set_gemm_mode(mode)
    try:
        got = ss.ss_decode_microbatch(gw, toks, offs, steps, limits)["tokens"]
        static = ss.ss_decode_microbatch_static(gw, toks, offs, steps, limits)["tokens"]
        assert np.array_equal(got, static)
        seqs = [np.concatenate([toks[i * plen:(i + 1) * plen], got[i, :-1]]) for i in range(rows)]
        forced = _forced(gw, seqs, [plen] * rows).reshape(rows, steps, shape.vocab)
        decided = 0
        for i in (0, rows // 2, rows - 1):
            ref = om.teacher_forced(seqs[i], first=plen - 1)
            assert np.abs(forced[i] - ref).max() <= TOL * np.abs(ref).max(), i
            top = np.partition(ref, -2, axis=-1)
            clear = top[:, -1] - top[:, -2] > 2 * TOL * np.abs(ref).max()
            assert np.array_equal(got[i][clear], ref.argmax(-1)[clear]), i
            decided += clear.sum()
        assert decided > steps
    finally:
        ss.ss_set_gemm_mode(0)
        gw.close()
