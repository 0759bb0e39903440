"""The gate/up projection of 65 to 128 rows by workgroups of seven and eight weight blocks, with a last workgroup that is full, partly
filled or of a single block, against the fp64 oracle; one, two and three chunks of K.

A weight block is one of a thousand and more whose products a row's feed-forward output sums, so rows of logits are compared in
their 2-norm.  What rounds on the way to them is the normed hidden state, the attention's output, the normed state of the feed-forward, its SwiGLU
products and the final norm: five values, each rounded to half once, by 2^-11 of itself at most, and fp32 sums.  The oracle without the
last block is at least three times that bound away, which the test makes sure of."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx, oracle_rollout, row_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,hidden", [(1600, 64), (1099, 256), (1100, 272), (2041, 64), (2001, 272)])
def test_gate_up_by_wide_workgroups(blocks, hidden):
    shape = synth.ModelShape(1, hidden, 1, 1, 64, 16 * blocks, 700)
    blob = synth.make_weights(shape, 4)
    rows = 70
    prompts, lens = synth.make_prompts(shape.vocab, rows, 3, seed=6)
    weights = synth.widen_to_f32(blob)
    ref = oracle_rollout(shape, weights, prompts, lens, G=1, max_new=3, temperature=1.0, seed=2, want_logits=True)
    ctx = make_ctx(shape, rows, 6, blob)
    out = ctx.rollout(prompts, lens, 1, 3, 1.0, 2, forced=ref["tokens"], want_logits=True)
    ctx.close()
    bound = 5 * 2.0 ** -11
    err = row_error(out["logits"], ref["logits"])
    print(f"row error {err:.2e}, bound {bound:.2e}")
    assert err < bound
    at, dims = synth.blob_offsets(shape)["layers.0.w_down"]
    short = np.array(weights).reshape(-1)
    short[at:at + dims[0] * dims[1]].reshape(dims)[:, -16:] = 0   # a block of 32 rows is 16 gates and their ups
    without = oracle_rollout(shape, short, prompts, lens, G=1, max_new=3, temperature=1.0, seed=2, forced=ref["tokens"], want_logits=True)
    assert row_error(without["logits"], ref["logits"]) > 3 * bound
