"""The all-fp32 path where some products of a step make their operand themselves (norm, SwiGLU) and others are too large for that, on either
side of the line for the feed-forward, the QKV projection and the lm_head, with rows that stop early, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import F32_LOGIT_TOL, F32_LOGPROB_TOL, check_tokens_fp32_sampler, make_ctx, oracle_rollout, valid_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,kv,ffn,vocab", [(256, 2, 2000, 3000), (256, 2, 2800, 700), (640, 8, 100, 900), (64, 1, 64, 12000)])
def test_products_on_either_side_of_the_line(hidden, kv, ffn, vocab):
    shape = synth.ModelShape(2, hidden, 2 * kv, kv, 64, ffn, vocab, dtype="fp32")
    blob = synth.make_weights(shape, 5, gain_jitter=0.1)
    prompts, lens = synth.make_prompts(shape.vocab, 3, 40, seed=4)
    stop = np.array([5, 1, 3, 5, 2, 4], np.int32)
    ref = oracle_rollout(shape, synth.widen_to_f32(blob), prompts, lens, G=2, max_new=5, temperature=1.0, seed=6, stop_lens=stop, want_logits=True)
    ctx = make_ctx(shape, 6, 45, blob)
    out = ctx.rollout(prompts, lens, 2, 5, 1.0, 6, stop_lens=stop, forced=np.maximum(ref["tokens"], 0), want_logits=True)
    mask = valid_mask(ref["lens"], 5)
    assert np.array_equal(out["lens"], ref["lens"])
    assert np.abs(out["logits"] - ref["logits"])[mask].max() < F32_LOGIT_TOL
    if check_tokens_fp32_sampler(out["tokens"], ref, mask) == 0:
        assert np.abs(out["logprobs"] - ref["logprobs"])[mask].max() < F32_LOGPROB_TOL
    ctx.close()


@pytest.mark.parametrize("qk_norm", [False, True])
def test_contexts_on_either_side_of_the_scores_that_fit(qk_norm):
    """The decode attention makes its own query and key only while they fit beside the scores of a full context: the same results either way."""
    shape = synth.TINY.replace(qk_norm=qk_norm)
    blob = synth.make_weights(shape, 3, gain_jitter=0.1)
    prompts, lens = synth.make_prompts(shape.vocab, 2, 33, seed=9)
    outs = []
    for max_ctx in (39, 15872, 15873, 16384):
        ctx = make_ctx(shape, 4, max_ctx, blob)
        outs.append(ctx.rollout(prompts, lens, 2, 6, 1.0, 2, want_logits=True))
        ctx.close()
    ref = oracle_rollout(shape, synth.widen_to_f32(blob), prompts, lens, G=2, max_new=6, temperature=1.0, seed=2, forced=outs[0]["tokens"], want_logits=True)
    assert np.abs(outs[0]["logits"] - ref["logits"]).max() < F32_LOGIT_TOL
    for out in outs[1:]:
        for k in ("tokens", "logprobs", "logits"):
            assert np.array_equal(out[k], outs[0][k])
