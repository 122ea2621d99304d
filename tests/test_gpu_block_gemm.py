"""The projections of prompt forwards at the edges of the block kernel's tiles, through whole forwards, against the
oracle: row counts around 16, 64, 128 and 256, widths that are no multiple of a tile (gate|up of 344 strips, a head of 65),
an odd number of k-blocks per slice.  Modes 0 and 1 take the tiles that the plan picks, the others force each of the fifteen
tiles on every projection: rotation and slots, residual sums, SwiGLU and plain sums, with k-slices (down) and without."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape("block", 1, 512, 4, 128, 2752, 1040)
# fp32 sums of products of halves: the oracle has exact weights and unrounded activations; one layer stays within 2e-3
# (a projection input is rounded once to 11 bits: 2^-12 relative per rounding, six of them and the cache's two)
TOL = 2e-3


@pytest.fixture(scope="module")
def model(oracle_built):
    W = synth.make_weights(SHAPE, seed=9, norm_jitter=0.1, threads=1)
    gw = ss.Weights(SHAPE, W)
    yield gw, OracleModel(SHAPE, W, "f32")
    gw.close()


@pytest.mark.parametrize("mode", [0, 1] + [1 + 16 * (t + 1) for t in range(5)])
@pytest.mark.parametrize("rows", [65, 127, 129, 145, 256, 257, 513, 895, 897, 1025])
def test_prompt_logits_match_the_oracle(model, rows, mode):
    gw, om = model
    rng = np.random.default_rng(rows)
    lens, left = [], rows
    while left > 0:
        n = int(min(left, rng.integers(20, 60)))
        lens.append(n)
        left -= n
    toks = rng.integers(0, SHAPE.vocab, rows).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ss.ss_set_gemm_mode(mode)
    try:
        got = ss.ss_forward_logits(gw, toks, offs, np.array(lens, np.int32), all_prompt_logits=True)
    finally:
        ss.ss_set_gemm_mode(0)
    for i in sorted({0, 1, len(lens) // 2, len(lens) - 1} & set(range(len(lens)))):
        ref = om.teacher_forced(toks[offs[i]:offs[i + 1]], first=0)
        err = np.abs(got[offs[i]:offs[i + 1]] - ref).max() / np.abs(ref).max()
        assert err <= TOL, (rows, mode, i, err)
    # every row is an independent sequence of sums: the same prompts alone give the same logits within rounding
    assert np.isfinite(got).all()


@pytest.mark.parametrize("tile", range(5, 15))
@pytest.mark.parametrize("rows", [65, 161, 193, 385, 641, 769])   # around the tiles' heights, one to eight of them
def test_prompt_logits_match_the_oracle_in_every_other_tile(model, rows, tile):
    test_prompt_logits_match_the_oracle(model, rows, 1 + 16 * (tile + 1))


@pytest.fixture(scope="module")
def many(model):
    """12311 token-rows, and their logits from forwards of a thirteenth of them each, where no die keeps row tiles of its own."""
    gw, _ = model
    rng = np.random.default_rng(12311)
    lens = rng.integers(20, 60, 400)
    lens = lens[:np.searchsorted(np.cumsum(lens), 12311) + 1].astype(np.int32)
    lens[-1] -= lens.sum() - 12311
    toks = rng.integers(0, SHAPE.vocab, 12311).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    parts = [ss.ss_forward_logits(gw, toks[offs[g[0]]:offs[g[-1] + 1]], offs[g[0]:g[-1] + 2] - offs[g[0]], lens[g], all_prompt_logits=True)
             for g in np.array_split(np.arange(len(lens)), 13)]
    return toks, offs, lens, np.concatenate(parts)


@pytest.mark.parametrize("tile", [None, 0, 1, 9, 13, 14])   # as chosen; every tile of 16 strips or more
def test_forwards_in_which_dies_keep_their_row_tiles(model, many, tile):
    # 49 tiles of 256 rows, 39 of 320, 33 of 384: 6, 4 and 4 for each die, and 1, 7 and 1 left over, the last of them not full
    gw, om = model
    toks, offs, lens, want = many
    ss.ss_set_gemm_mode(0 if tile is None else 1 + 16 * (tile + 1))
    try:
        got = ss.ss_forward_logits(gw, toks, offs, lens, all_prompt_logits=True)
    finally:
        ss.ss_set_gemm_mode(0)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    for i in (0, len(lens) // 2, len(lens) - 1):
        ref = om.teacher_forced(toks[offs[i]:offs[i + 1]], first=0)
        assert np.abs(got[offs[i]:offs[i + 1]] - ref).max() <= TOL * np.abs(ref).max(), (tile, i)
