"""A continuous rollout whose records are long and end together: more records at a time than the pinned buffer of the hand-over holds
(4 MiB; 131 KB a record here, so 32), both when they are handed over and when the next ones are opened with forced tokens."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [40, 33, 1])
def test_long_records_that_end_together(slots):
    shape = synth.TINY
    max_new, P = 8192, 80
    blob = synth.make_weights(shape, 0)
    prompts, lens = synth.make_prompts(shape.vocab, P, 6, seed=1)
    stop = np.full(P, 3, np.int32)
    stop[::7] = 2
    forced = np.random.default_rng(2).integers(0, shape.vocab, size=(P, max_new)).astype(np.int32)
    ref_ctx = make_ctx(shape, P, 6 + 3, blob)
    ref = ref_ctx.rollout(prompts, lens, 1, 3, 1.0, 4, stop_lens=stop, forced=np.ascontiguousarray(forced[:, :3]))
    ref_ctx.close()
    ctx = make_ctx(shape, slots, 6 + max_new, blob)
    out = ctx.rollout(prompts, lens, 1, max_new, 1.0, 4, stop_lens=stop, forced=forced, continuous=True)
    ctx.close()
    assert np.array_equal(out["lens"], stop)
    assert np.array_equal(out["tokens"][:, :3], ref["tokens"])
    assert np.array_equal(out["versions"][:, :3], ref["versions"])
    assert np.abs(out["logprobs"][:, :3] - ref["logprobs"]).max() < 1e-5     # other summation orders of fp32 attention and norm
    assert (out["tokens"][:, 3:] == -1).all() and (out["logprobs"][:, 3:] == 0).all() and (out["versions"][:, 3:] == -1).all()
