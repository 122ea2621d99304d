"""Decode forwards of one to four rows run kernels of their own (norms inside the projections).  A row's logits are the same
numbers, bit for bit, as in a forward of more rows, where the other kernels run: whoever else is still alive does not matter."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu

# d_model, heads, head_dim, ffn, vocab: sweep and skinny kernels at 16 rows, one and two waves per unit, k-slices that divide the groups
# of 4 k-blocks and that do not, chains of quarters in waves of their own and in one wave, more than 4096 columns
SHAPES = [(4096, 32, 128, 11008, 32000), (5120, 40, 128, 13824, 8000), (2048, 16, 128, 5504, 16000), (1024, 16, 64, 2816, 4000),
          (3072, 24, 128, 8192, 4000), (1152, 9, 128, 3200, 1040), (8192, 64, 128, 1664, 1040), (640, 10, 64, 16384, 528)]


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[3]}")
def test_logits_are_those_of_a_forward_of_more_rows(shape, rows):
    d, heads, hd, ffn, vocab = shape
    model = synth.ModelShape("few", 1, d, heads, hd, ffn, vocab)
    rng = np.random.default_rng(rows)
    W = synth.make_weights(model, seed=11, norm_jitter=0.2, threads=8)
    gw = ss.Weights(model, W)
    B, plen, steps = 6, 5, 3
    toks = [rng.integers(0, vocab, plen + steps).astype(np.int32) for _ in range(B)]

    def run(keep):   # `keep` rows decode all steps, the others end with their prompts
        seqs = [t if i < keep else t[:plen] for i, t in enumerate(toks)]
        offs = np.concatenate([[0], np.cumsum([len(q) for q in seqs])]).astype(np.int32)
        out = ss.ss_forward_logits(gw, np.concatenate(seqs), offs, np.full(B, plen, np.int32))
        return out[:rows * (steps + 1)]

    few, many = run(rows), run(B)
    gw.close()
    assert np.array_equal(few, many)
    ref = OracleModel(model, W, "f32").teacher_forced(toks[0], first=plen - 1)
    assert np.abs(few[:steps + 1] - ref).max() <= 2e-3 * np.abs(ref).max()
