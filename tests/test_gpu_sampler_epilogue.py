"""The sampler fused into the lm_head against the fp32 sampler over the materialised logits of the same step: tokens must be the
same everywhere (both decide by the same fp32 scores; the logits are bit-identical), log-probs within fp32 rounding.
Vocabularies that end inside a weight block, inside a wavefront's share and on the first entry of a strip; every launch form by
batch size; temperatures at which the scores span thousands and at which they are nearly all noise."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [3, 40, 70, 130, 260])
@pytest.mark.parametrize("vocab", [1000, 2049, 4099])
def test_fused_sampler_takes_the_tokens_of_the_fp32_sampler(rows, vocab):
    shape = synth.ModelShape(1, 256, 4, 2, 64, 512, vocab)
    blob = synth.make_weights(shape, 5)
    prompts, lens = synth.make_prompts(vocab, rows, 5, seed=rows, ragged=True)
    prompts = np.maximum(prompts, 0)
    new = 6
    forced = np.random.default_rng(vocab).integers(0, vocab, size=(rows, new)).astype(np.int32)
    ctx = make_ctx(shape, rows, 5 + new, blob)
    for temperature in (1.0, 1e-3, 60.0):
        a = ctx.rollout(prompts, lens, 1, new, temperature, 9, forced=forced)
        b = ctx.rollout(prompts, lens, 1, new, temperature, 9, forced=forced, unfused_sampler=True)
        assert np.array_equal(a["tokens"], b["tokens"]), temperature
        # both sum a few thousand fp32 exponentials and round z and log-sum-exp (up to 2000 at T = 1e-3) to fp32
        z = np.abs(b["logprobs"]).max() + 0.1 / temperature
        assert np.abs(a["logprobs"] - b["logprobs"]).max() < 2e-6 * max(8.0, z), temperature
    ctx.close()
