"""The two main loops of the LDS-ring GEMM sum in the same bits: the same strings, scored in a batch whose projections take 256 x 256 tiles (16 x 16 x 32 MFMAs,
by pairs of k-steps) and in a smaller one where they take 256 x 128 tiles (32 x 32 x 16), have equal log-probs.

A string's last bits depend on nothing else here: its attention blocks and norms are its own, the lm_head takes the same tiles in both batches, and every projection is
cut over K alike.  Sums in another order differ in their last bits, by some 1e-7, and a half behind them (2^-11) then rounds the other way once in some thousand: every
row or two of a thousand features, and fp32 log-probs with it."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx

pytestmark = pytest.mark.gpu

LENGTH = 257   # 256 rows a string


@pytest.mark.parametrize("shape,few", [
    # gate/up alone changes its tiles (9 strips x 16 row blocks against 9 x 2); the down projection is cut in two in both batches, and the small one's
    # QKV projection has its norm and rotation in a kernel of their own
    (synth.ModelShape(1, 384, 4, 2, 64, 1040, 500), 2),
    # all four projections do, uncut in both: 8 or 9 strips x 16 row blocks against x 12; QKV with its epilogue, heads of 128 with and without a norm
    (synth.ModelShape(1, 2048, 8, 4, 128, 1040, 500), 12),
    (synth.ModelShape(1, 2048, 8, 4, 128, 1040, 500, qk_norm=True), 12),
    # heads of 64; QKV 60 weight blocks in eight strips, so the last strip has four past the end
    (synth.ModelShape(1, 1920, 20, 5, 64, 1168, 500, qk_norm=True), 12),
])
def test_both_loops_in_the_same_bits(shape, few):
    blob = synth.make_weights(shape, 6)
    toks = np.random.default_rng(few).integers(0, shape.vocab, size=(16, LENGTH)).astype(np.int32)
    ctx = make_ctx(shape, 16, LENGTH, blob)
    many = ctx.logprobs(toks, np.full(16, LENGTH, np.int32), 1.0)
    some = ctx.logprobs(toks[:few], np.full(few, LENGTH, np.int32), 1.0)
    ctx.close()
    assert np.abs(many[:, 1:]).min() > 0.0
    assert np.array_equal(many[:few], some), np.argwhere(many[:few] != some)[:5]
