"""Micro-batches of a group that share their decode forwards: every token is the one that the micro-batch gets alone.  Random
weights, so that most choices are near ties and a changed sum shows; widths on both sides of what the small-batch projection
kernels and the attention's shapes are chosen by, with the 12-bit weight copies and without."""
import numpy as np
import pytest

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = {
    "7b": synth.LLAMA7B.with_layers(2),                                      # o in the skinny kernel, the rest in the sweep kernel
    "40 heads": synth.ModelShape("h40", 2, 5120, 40, 128, 6912, 4096),       # 8 attention waves up to 12 rows, 4 above
    "d2048": synth.ModelShape("d2048", 2, 2048, 32, 64, 5504, 4096),         # most in the skinny kernel; heads of 64
}
COUNTERS = ("steps", "padded_row_steps", "computed_row_steps", "n_failed", "useful_tokens", "n_mb_first", "n_mb_failure",
            "prompt_tokens")


@pytest.fixture(scope="module", params=sorted(SHAPES))
def model(request):
    shape = SHAPES[request.param]
    gw = ss.Weights(shape, synth.make_weights(shape, seed=3, threads=8))
    yield shape, gw
    gw.close()


# micro-batches of 16, of 1 to 5, of sizes on both sides of a strip (variable batch sizes), a last one of a few rows; prompts
# that make some micro-batches too long for a strip's attention plan
@pytest.mark.parametrize("flags,batch,plen,copies", [((), 16, 30.0, 1), (("SORT", "BIN", "FCR"), 16, 30.0, 0),
                                                      (("SORT", "BIN", "FCR", "COMPACT"), 5, 120.0, 1),
                                                      (("SORT", "BIN", "FCR", "VBS", "COMPACT"), 8, 30.0, 1)])
def test_tokens_and_counters_are_those_of_one_at_a_time(model, flags, batch, plen, copies):
    shape, gw = model
    w = synth.make_group(shape, 75, 91, ("lognormal", plen, 0.6, 4, 600), ("lognormal", 12.0, 0.7, 1, 40), 0.3, 40, 8, flags,
                         base_batch=batch, max_batch=48)
    pol = ss.make_policy(flags, batch, 40, 48)
    preds = w.pred_lens if flags else None
    gw.set_option(ss.SS_OPT_WEIGHT_COPIES, copies)
    try:
        got = {}
        for lanes in (1, 4, 3, 2):
            gw.set_option(ss.SS_OPT_IN_FLIGHT, lanes)
            r = got[lanes] = ss.ss_run_group(gw, w.prompt_tokens, w.prompt_offsets, w.target_lens, preds, 8 if flags else 0, pol)
            assert np.array_equal(r["tokens"], got[1]["tokens"]), lanes
            assert np.array_equal(r["lens"], w.target_lens), lanes
            for name in COUNTERS:
                assert r["stats"][name] == got[1]["stats"][name], (lanes, name)
    finally:
        gw.set_option(ss.SS_OPT_IN_FLIGHT, ss.SS_IN_FLIGHT_DEFAULT)
        gw.set_option(ss.SS_OPT_WEIGHT_COPIES, 1)


@pytest.mark.parametrize("seed", [2, 3])
def test_a_member_that_ends_early_leaves_the_others_their_sums(model, seed):
    """Two micro-batches of 4 rows, few enough for 16 attention waves where a context is long enough, which neither's is: a long
    prompt that ends early and a short one that runs on.  The first one's prompt does not count once it has ended."""
    shape, gw = model
    limit = 64 * 512 // shape.head_dim   # the longest context of 8 waves
    rng = np.random.default_rng(seed)
    plens = [limit - 56] * 4 + [16] * 4
    targets = np.array([48] * 4 + [limit - 24] * 4, np.int32)
    toks = rng.integers(0, shape.vocab, sum(plens)).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(plens)]).astype(np.int32)
    pol = ss.make_policy(("SORT", "BIN", "FCR"), 4, limit - 24, 16)
    try:
        got = []
        for lanes in (1, 4):
            gw.set_option(ss.SS_OPT_IN_FLIGHT, lanes)
            r = ss.ss_run_group(gw, toks, offs, targets, targets, 8, pol)
            assert r["stats"]["n_mb_first"] == 2 and r["stats"]["n_failed"] == 0
            got.append(r["tokens"])
        assert np.array_equal(got[0], got[1])
    finally:
        gw.set_option(ss.SS_OPT_IN_FLIGHT, ss.SS_IN_FLIGHT_DEFAULT)
