"""The query operand of the prompt attention keeps the bits that the decode attention's fp32 dot product sees.  Small
queries against large keys: an error of a query element moves a score by that error times a key of 2e4.  The last
position of a sequence is computed once by the prompt forward and once by a decode step on the same slots."""
import numpy as np
import pytest

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

# A query element is the sum of two halves, so below 1/8 it is held to a multiple of 2^-24: an error of 2^-24 / sqrt(12),
# times the 128 elements' root, a key of 2e4 and 1/sqrt(128), is 3.4e-4 of a score, the relative error of a probability.
# Probabilities and the two projection inputs behind them are rounded to 11 bits, 2^-11 / sqrt(12) = 1.4e-4 each: in all
# 4.2e-4 in the 2-norm, a little less where a softmax is dominated by few slots.  A query scaled by log2(e)/sqrt(128)
# before it is split has 7.8 times the first error, 2.7e-3.
TOL = 1e-3


@pytest.mark.parametrize("head_dim", [64, 128])
def test_prompt_and_decode_see_the_same_query(head_dim):
    shape = synth.ModelShape("qbits", 1, 512, 512 // head_dim, head_dim, 256, 512)
    W = synth.make_weights(shape, seed=77, threads=1)
    names = [n for n, _ in shape.tensor_specs()]

    def scaled(name, std):
        i = names.index(name)
        W[i] = synth.f32_to_bf16_bits(synth.bf16_bits_to_f32(W[i]) * np.float32(std / 0.02))

    scaled("embed", 1.0)
    scaled("l0.wk", 2.0e4 / 512 ** 0.5)        # keys of 2e4, three deviations inside the half range
    scaled("l0.wq", 1.0e-4 / 512 ** 0.5)       # scores of a few units
    scaled("l0.wv", 1.0)
    scaled("l0.wo", 1.0)                       # the attention's share of the residual stream dwarfs the embedding's
    scaled("l0.wd", 0.0)
    rng = np.random.default_rng(5)
    rows, n = 32, 61
    toks = rng.integers(0, shape.vocab, (rows, n)).astype(np.int32)
    offs = (np.arange(rows + 1) * n).astype(np.int32)
    gw = ss.Weights(shape, W)
    try:
        prompt = ss.ss_forward_logits(gw, toks.ravel(), offs, np.full(rows, n, np.int32)).astype(np.float64)
        step = ss.ss_forward_logits(gw, toks.ravel(), offs, np.full(rows, n - 1, np.int32))[1::2].astype(np.float64)
    finally:
        gw.close()
    err = np.linalg.norm(prompt - step) / np.linalg.norm(step)
    print(f"head_dim {head_dim}: prompt against decode {err:.2e}")
    assert err <= TOL, err
