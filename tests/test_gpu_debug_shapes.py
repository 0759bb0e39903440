"""The all-fp32 path at widths that are and are not multiples of four (vector and scalar loads of the same kernels), with fp32 and with
bf16 weights, prompts of one and of several tokens, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import F32_LOGIT_TOL, F32_LOGPROB_TOL, check_tokens_fp32_sampler, make_ctx, oracle_rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden,heads,kv,hd,ffn", [(250, 3, 3, 10, 70), (4, 1, 1, 2, 4), (260, 4, 2, 12, 516), (64, 2, 1, 66, 130), (96, 2, 2, 160, 64)])
def test_fp32_path_at_odd_widths(dtype, hidden, heads, kv, hd, ffn):
    shape = synth.ModelShape(2, hidden, heads, kv, hd, ffn, 301, dtype=dtype, qk_norm=hd > 60)
    blob = synth.make_weights(shape, 3, gain_jitter=0.1)
    prompts, lens = synth.make_prompts(shape.vocab, 3, 90, seed=2, ragged=True)
    lens[0] = 1
    prompts = np.maximum(prompts, 0)
    ref = oracle_rollout(shape, synth.widen_to_f32(blob), prompts, lens, G=2, max_new=5, temperature=1.0, seed=6, want_logits=True)
    ctx = make_ctx(shape, 6, 95, blob, debug_naive=dtype == "bf16")
    out = ctx.rollout(prompts, lens, 2, 5, 1.0, 6, forced=ref["tokens"], want_logits=True)
    assert np.abs(out["logits"] - ref["logits"]).max() < F32_LOGIT_TOL
    if check_tokens_fp32_sampler(out["tokens"], ref) == 0:
        assert np.abs(out["logprobs"] - ref["logprobs"]).max() < F32_LOGPROB_TOL
    ctx.close()
