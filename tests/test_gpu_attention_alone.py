"""Decode attention of small batches on either side of the lines between one workgroup of eight wavefronts per row and KV head and
splits over the keys: key counts around 1024 and 2048, batches that would take ten, five, two splits and one, one key, tails of a tile, against the
fp64 oracle.

A key is one of up to 2048 that a row's output averages, so the output projection is large here (the attention's output outweighs the
embedding in the residual stream) and rows of logits are compared in their 2-norm.  Nine values are rounded to half on the way to
them, by 2^-11 of themselves at most: normed state, query, key, value, weight of a key, attention output, the feed-forward's normed state and products, final
norm.  The oracle with one key exchanged is twice that bound away, which the test makes sure of."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx, oracle_rollout, row_error
from test_gpu_refused_calls import child  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv,hd,prompts,G,plen,new", [
    (2, 64, 1, 1, 1, 40),         # from one key on
    (2, 128, 1, 1, 1018, 7),      # 1024 keys: alone
    (2, 128, 1, 1, 1019, 7),      # 1025: split
    (8, 64, 4, 2, 1021, 5),       # 10 splits by the batch, 1025 keys
    (8, 64, 4, 4, 2041, 8),       # 5 splits by the batch, 2048 keys: alone
    (8, 64, 4, 4, 2042, 8),       # 2049: split
    (8, 128, 4, 8, 70, 5),        # 32 rows, two splits by the batch: alone whatever the keys
    (8, 64, 20, 2, 33, 5),        # 40 rows
    (8, 64, 41, 1, 33, 5),        # 41 rows fill the chip
])
def test_keys_and_batches_around_the_lines(kv, hd, prompts, G, plen, new):
    shape = synth.ModelShape(1, 128, 2 * kv, kv, hd, 64, 300)
    blob = synth.make_weights(shape, 3, gain_jitter=0.1).clone()
    at, dims = synth.blob_offsets(shape)["layers.0.wo"]
    blob[at:at + dims[0] * dims[1]] *= 64
    weights = synth.widen_to_f32(blob)
    toks, lens = synth.make_prompts(shape.vocab, prompts, plen, seed=2)
    N = prompts * G
    forced = np.random.default_rng(5).integers(0, shape.vocab, (N, new)).astype(np.int32)
    ctx = make_ctx(shape, N, plen + new, blob)
    out = ctx.rollout(toks, lens, G, new, 1.0, 6, forced=forced, want_logits=True)
    ctx.close()

    def oracle_logits(p, G, toks):
        return oracle_rollout(shape, weights, toks[p:p + 1], lens[p:p + 1], G=G, max_new=new, temperature=1.0, seed=6, forced=forced[p * G:(p + 1) * G],
                              want_logits=True)["logits"]

    bound = 9 * 2.0 ** -11
    for p in (0, prompts - 1):   # first and last group
        ref = oracle_logits(p, G, toks)
        err = row_error(out["logits"][p * G:(p + 1) * G], ref)
        print(f"row error {err:.2e}, bound {bound:.2e}")
        assert err < bound, p
        if p == 0:
            other = toks.copy()
            other[0, plen // 2] = (other[0, plen // 2] + 7) % shape.vocab
            assert row_error(oracle_logits(0, 1, other), ref[:1]) > 2 * bound


def test_how_many_workgroups_take_a_row(child):
    """Rows of as many keys as the longest one comes to (the last drawn token is no key): 1024 and 1025 with ten splits and more by the
    batch, 2048 and 2049 with five."""
    child("""
def splits(kv, rows, keys, continuous):
    s = synth.ModelShape(1, 64, kv, kv, 64, 64, 300)
    ctx = make_ctx(s, rows, keys + 8, synth.make_weights(s, 3))
    p, l = synth.make_prompts(s.vocab, 1, keys - 1, seed=2)
    shim.hip_refuse(b"attn_splitk_kernel", 1 << 30)
    ctx.rollout(p, l, rows, 2, 1.0, 6, continuous=continuous)
    assert shim.hip_seen() > 0
    ctx.close()
    return shim.hip_seen_grid()

want = {(2, 1): [(2, 1), (1024, 1), (1025, 32)], (8, 8): [(1024, 1), (1025, 10)], (8, 16): [(1025, 1), (2048, 1), (2049, 5)], (8, 32): [(3000, 1)]}
wrong = [(kv, rows, keys, n, got, continuous) for (kv, rows), lines in want.items() for keys, n in lines for continuous in (False, True)
         for got in [splits(kv, rows, keys, continuous)] if got != n]
print(wrong or "as expected")
""")
