"""The 12-bit copies of the weights (what decode batches stream) hold the same values as the halves they replace: two
models whose heads differ in one value of one row, so that one has such a copy and the other (0.5 has no 12-bit form) has
not, give the same numbers in every other column.  The copy carries eight times the weight, so weights that are subnormal
as halves are normal there, and the matrix unit may round a sum that contains one differently in its last bit: fewer than
one column in a thousand, by no more than an fp32 rounding of the largest partial sum.  A wrong weight changes every row
of its column by far more than that."""
import numpy as np
import pytest

from oracle.model_oracle import OracleModel
from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

pytestmark = pytest.mark.gpu


def _wide_head(shape, rng):
    """bf16 patterns over everything the 12-bit form covers: both zeros, all exponents below 2^-2, all mantissas, and the
    values below 2^-17 that are held as multiples of 2^-24."""
    v, d = shape.vocab, shape.d_model
    exp = rng.integers(0, 125, (v, d))                   # biased exponent 124 = [2^-3, 2^-2)
    exp = np.where(rng.random((v, d)) < 0.7, rng.integers(105, 125, (v, d)), exp)
    return ((rng.integers(0, 2, (v, d)) << 15) | (exp << 7) | rng.integers(0, 128, (v, d))).astype(np.uint16)


@pytest.mark.parametrize("mode", [5, 6])                 # skinny kernel; sweep kernel, one wave per unit in both forms
@pytest.mark.parametrize("rows", [1, 16, 17, 48, 96, 97])
def test_logits_are_the_same_with_and_without_the_12_bit_copy(mode, rows):
    shape = synth.ModelShape("narrow", 1, 512, 4, 128, 640, 1040)
    rng = np.random.default_rng(rows)
    W = synth.make_weights(shape, seed=3, threads=1)
    W[-1] = _wide_head(shape, rng)
    other = list(W)
    other[-1] = W[-1].copy()
    other[-1][1039, 5] = synth.f32_to_bf16_bits(np.array([0.5], np.float32))[0]
    toks = rng.integers(0, shape.vocab, rows * 3).astype(np.int32)
    offs = np.arange(rows + 1, dtype=np.int32) * 3
    ss.ss_set_gemm_mode(mode)
    try:
        out = []
        for weights in (W, other):
            gw = ss.Weights(shape, weights)
            out.append(ss.ss_forward_logits(gw, toks, offs, np.full(rows, 1, np.int32)))   # a prompt forward, two steps
            gw.close()
    finally:
        ss.ss_set_gemm_mode(0)
    assert np.isfinite(out[0]).all()
    a, b = out[0][:, :1039], out[1][:, :1039]
    assert (a != b).mean() < 1e-3
    assert np.abs(a - b).max() <= 2.0 ** -22 * np.abs(a).max()
    assert not np.array_equal(out[0][:, 1039], out[1][:, 1039])


@pytest.mark.parametrize("rows", [1, 16, 17, 48, 96])
@pytest.mark.parametrize("mode", [0, 1, 2, 6])           # as chosen; skinny; sweep, two waves per unit and one
def test_sliced_projections_agree_with_and_without_the_copies(mode, rows):
    """The same handle with its copies and without, where k is cut in slices and shared by waves that do not divide it
    (22 and 86 groups of 4 k-blocks; the two forms add up in different orders), and against the oracle."""
    shape = synth.ModelShape("sliced", 1, 2816, 22, 128, 11008, 272)
    rng = np.random.default_rng(rows)
    W = synth.make_weights(shape, seed=3, threads=8)
    toks = rng.integers(0, shape.vocab, rows * 4).astype(np.int32)
    offs = np.arange(rows + 1, dtype=np.int32) * 4
    gw = ss.Weights(shape, W)
    ss.ss_set_gemm_mode(mode)
    try:
        out = []
        for copies in (1, 0):
            gw.set_option(ss.SS_OPT_WEIGHT_COPIES, copies)
            out.append(ss.ss_forward_logits(gw, toks, offs, np.full(rows, 1, np.int32)))   # a prompt forward, three steps
    finally:
        ss.ss_set_gemm_mode(0)
        gw.close()
    # fp32 sums in another order move a projection input to the neighbouring half now and then (2^-11 of an element)
    assert np.abs(out[0] - out[1]).max() <= 1e-3 * np.abs(out[1]).max()
    om = OracleModel(shape, W, "f32")
    for i in sorted({0, rows // 2, rows - 1}):
        ref = om.teacher_forced(toks[offs[i]:offs[i + 1]], first=0)
        for o in out:
            assert np.abs(o[4 * i:4 * i + 4] - ref).max() <= 2e-3 * np.abs(ref).max(), (mode, rows, i)


@pytest.mark.parametrize("rows", [1, 17])
@pytest.mark.parametrize("ffn", [1280, 4096, 5120, 10240, 10368])   # strips of 30, 96, 120, 240 and 243 KiB: with a gap after them or none
def test_strips_with_gaps_agree_with_and_without_the_copies(ffn, rows):
    shape = synth.ModelShape("gaps", 1, 512, 4, 128, ffn, 272)
    rng = np.random.default_rng(rows)
    W = synth.make_weights(shape, seed=5, threads=8)
    toks = rng.integers(0, shape.vocab, rows * 3).astype(np.int32)
    offs = np.arange(rows + 1, dtype=np.int32) * 3
    gw = ss.Weights(shape, W)
    out = []
    for copies in (1, 0):
        gw.set_option(ss.SS_OPT_WEIGHT_COPIES, copies)
        out.append(ss.ss_forward_logits(gw, toks, offs, np.full(rows, 1, np.int32)))
    gw.close()
    # as above: an input moved to the neighbouring half now and then
    assert np.abs(out[0] - out[1]).max() <= 1e-3 * np.abs(out[1]).max()
    ref = OracleModel(shape, W, "f32").teacher_forced(toks[:3], first=0)
    assert np.abs(out[0][:3] - ref).max() <= 2e-3 * np.abs(ref).max()


def test_read_probe_reads_what_small_batches_stream():
    """The probe that the projections are compared with: three quarters of the bytes where a matrix has its copy."""
    shape = synth.ModelShape("probe", 1, 1024, 8, 128, 2048, 4096)      # every matrix whole 64 KiB chunks in both forms
    W = synth.make_weights(shape, seed=3, threads=8)
    halves = (4 * 1024 * 1024 + 3 * 1024 * 2048 + 4096 * 1024) * 2
    W[-1][5, 5] = synth.f32_to_bf16_bits(np.array([0.5], np.float32))[0]   # the head has no copy
    gw = ss.Weights(shape, W)
    head = 4096 * 1024 * 2
    assert ss.ss_bench_read_stream(gw, 2)[1] == (halves - head) * 3 // 4 + head
    gw.set_option(ss.SS_OPT_WEIGHT_COPIES, 0)
    assert ss.ss_bench_read_stream(gw, 2)[1] == halves
    for rows in (16, 200):
        ms, launches = ss.ss_bench_weight_stream(gw, rows, 2)
        assert launches == 5 and (ms > 0).all()
    gw.close()
