"""The gate/up projection of 65 to 128 rows by workgroups of seven and eight weight blocks, with a last workgroup that is full, partly
filled or of a single block, against the fp64 oracle; one, two and three chunks of K."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import BF16_LOGIT_TOL, make_ctx, oracle_rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,hidden", [(1600, 64), (1099, 256), (1100, 272), (2041, 64), (2001, 272)])
def test_gate_up_by_wide_workgroups(blocks, hidden):
    shape = synth.ModelShape(1, hidden, 1, 1, 64, 16 * blocks, 700)
    blob = synth.make_weights(shape, 4)
    rows = 70
    prompts, lens = synth.make_prompts(shape.vocab, rows, 3, seed=6)
    ref = oracle_rollout(shape, synth.widen_to_f32(blob), prompts, lens, G=1, max_new=3, temperature=1.0, seed=2, want_logits=True)
    ctx = make_ctx(shape, rows, 6, blob)
    out = ctx.rollout(prompts, lens, 1, 3, 1.0, 2, forced=ref["tokens"], want_logits=True)
    assert np.abs(out["logits"] - ref["logits"]).max() < BF16_LOGIT_TOL
    ctx.close()
