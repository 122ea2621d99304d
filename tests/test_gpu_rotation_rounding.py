"""A prompt's keys and queries do not depend on the kernel that rotates them: with few token-rows the k-slices of q|k|v are
summed and rotated by a launch of their own, with many the projection rotates its own sums.  Every row of every matrix here has
one weight, a power of two, so that all sums of products are exact in any order and whole forwards agree bit for bit.  Large weights of
q, k and o make scores, and with them the logits, follow a key that is rounded to the neighbouring half."""
import numpy as np
import pytest

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu


def _one_weight_a_row(shape, seed):
    rng = np.random.default_rng(seed)
    out = []
    for name, shp in shape.tensor_specs():
        if name == "embed":
            w = rng.standard_normal(shp)
        elif len(shp) == 1:
            w = 1 + 0.1 * rng.standard_normal(shp)
        else:
            w = np.zeros(shp)
            size = {"wq": 2.0, "wk": 2.0, "wo": 8.0}.get(name.split(".")[-1], 1.0)
            w[np.arange(shp[0]), rng.permutation(max(shp))[:shp[0]] % shp[1]] = size * rng.choice([-1, 1], shp[0])
        out.append(synth.f32_to_bf16_bits(w.astype(np.float32)))
    return out


@pytest.mark.parametrize("hd", [64, 128])
def test_prompts_are_rotated_alike_in_small_and_large_forwards(hd):
    shape = synth.ModelShape("rotate", 2, 512, 512 // hd, hd, 640, 528)
    gw = ss.Weights(shape, _one_weight_a_row(shape, 7))
    rng = np.random.default_rng(hd)
    for mode in [0] + [1 + 16 * (t + 1) for t in range(15)] * 2:   # every tile of the block kernel
        lens = np.array([13, 29, 22] + [60] * 5, np.int32)         # 64 token-rows: rotated apart; 364: in the projection
        toks = rng.integers(0, shape.vocab, int(lens.sum())).astype(np.int32)
        offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        few = ss.ss_forward_logits(gw, toks[:64], offs[:4], lens[:3], all_prompt_logits=True)
        ss.ss_set_gemm_mode(mode)
        try:
            many = ss.ss_forward_logits(gw, toks, offs, lens, all_prompt_logits=True)
        finally:
            ss.ss_set_gemm_mode(0)
        assert np.isfinite(few).all() and np.abs(few).max() > 0.01
        assert np.array_equal(few, many[:64]), mode
    gw.close()
