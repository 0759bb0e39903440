"""Decode attention of small batches on either side of the lines between one workgroup of eight wavefronts per row and KV head and
splits over the keys: key counts around 1024 and 2048, batches that would take ten, five, two splits and one, one key, tails of a tile, against the
fp64 oracle."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import BF16_LOGIT_TOL, make_ctx, oracle_rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv,hd,prompts,G,plen,new", [
    (2, 64, 1, 1, 1, 40),         # from one key on
    (2, 128, 1, 1, 1017, 7),      # 1024 keys: alone
    (2, 128, 1, 1, 1018, 7),      # 1025: split
    (8, 64, 4, 2, 1020, 5),       # 10 splits by the batch, 1025 keys
    (8, 64, 4, 4, 2040, 8),       # 5 splits by the batch, 2048 keys: alone
    (8, 64, 4, 4, 2043, 8),       # 2051: split
    (8, 128, 4, 8, 70, 5),        # 32 rows, two splits by the batch: alone whatever the keys
    (8, 64, 20, 2, 33, 5),        # 40 rows
    (8, 64, 41, 1, 33, 5),        # 41 rows fill the chip
])
def test_keys_and_batches_around_the_lines(kv, hd, prompts, G, plen, new):
    shape = synth.ModelShape(1, 128, 2 * kv, kv, hd, 64, 300)
    blob = synth.make_weights(shape, 3, gain_jitter=0.1)
    toks, lens = synth.make_prompts(shape.vocab, prompts, plen, seed=2)
    N = prompts * G
    forced = np.random.default_rng(5).integers(0, shape.vocab, (N, new)).astype(np.int32)
    ctx = make_ctx(shape, N, plen + new, blob)
    out = ctx.rollout(toks, lens, G, new, 1.0, 6, forced=forced, want_logits=True)
    ctx.close()
    for p in (0, prompts - 1):   # first and last group
        rows = slice(p * G, (p + 1) * G)
        ref = oracle_rollout(shape, synth.widen_to_f32(blob), toks[p:p + 1], lens[p:p + 1], G=G, max_new=new, temperature=1.0, seed=6, forced=forced[rows],
                             want_logits=True)
        assert np.abs(out["logits"][rows] - ref["logits"]).max() < BF16_LOGIT_TOL, p
