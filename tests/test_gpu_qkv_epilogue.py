"""What the QKV projection of a large pass leaves in the cache when it rotates and appends in its own epilogue, bit for bit: both tile
forms, both head dims, head counts that no tile divides, sequences that start and end inside a block of 32 rows, sequences of one row,
a pass that goes on in the middle of a sequence, rows that have ended.  The value projection repeats the key projection's one-hot rows, so cached
values are the keys before norm and rotation (exact in half precision), at the places that the cache's form gives them."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx
from test_gpu_qkv_post import F32, expected_keys, tiles
from test_gpu_refused_calls import child  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


def one_hot_keys_and_values(shape, r):
    """(blob, embedding, columns): the key and the value projection are the same one-hot rows, at `columns` of the hidden state."""
    blob = synth.make_weights(shape, 3).clone()
    at = 0
    for name, dims, _ in synth.tensor_table(shape):
        n = int(np.prod(dims))
        if name.endswith(("wk", "wv")):
            w = blob[at:at + n].view(*dims)
            w.zero_()
            cols = r.integers(0, shape.hidden, dims[0]) if name.endswith("wk") else cols
            w[np.arange(dims[0]), cols] = 1.0
        elif name.endswith("embed"):
            embed = blob[at:at + n].view(*dims).float().numpy()
        at += n
    return blob, embed, cols


def check_cache(shape, ctx, before, tokens, lens, max_ctx, embed, cols):
    """The cache slot of sequence n holds tokens[n, :lens[n]] and nothing behind them."""
    base, kv, hd = (-ctx.arena.data_ptr()) % 256, shape.n_kv_heads, shape.head_dim
    # the cache is the first part of the arena, behind the weights, that a pass writes
    start = int((ctx.arena[base:] != before).nonzero()[0, 0]) // 256 * 256
    nt = (max_ctx + 31) // 32
    raw = ctx.arena[base + start:base + start + len(lens) * kv * nt * 64 * hd * 2].cpu().numpy().view(np.float16).reshape(len(lens), kv, nt, 64 * hd)
    for n, length in enumerate(lens):
        k, v = tiles(raw[n], hd)
        assert (k[:, length:] == 0).all() and (v[:, length:] == 0).all(), n
        k, v = k[:, :length], v[:, :length].astype(F32)
        # the values are the normed embedding at the one-hot columns, to within a rounding of half
        x = embed[tokens[n, :length]]
        x = (x / np.sqrt((x.astype(np.float64) ** 2).mean(-1, keepdims=True) + shape.rms_eps))[:, cols].reshape(length, kv, hd).transpose(1, 0, 2)
        assert np.abs(v - x).max() <= 2.0 ** -10 * np.abs(x).max(), n
        want, _ = expected_keys(v, shape.rope_base, shape.rms_eps if shape.qk_norm else None, True)
        assert np.array_equal(k, want), (n, int((k != want).sum()))


def arena_now(ctx):
    return ctx.arena[(-ctx.arena.data_ptr()) % 256:].clone()


@pytest.mark.parametrize("hd,kv,H,lens", [
    (64, 3, 512, [250, 2, 33, 260, 3, 9, 300, 257, 64, 65, 700, 380]),             # 2311 rows, 18 weight blocks: 50 tiles of 256 x 128
    (128, 3, 512, [251, 3, 2, 280, 34, 10, 299, 258, 66, 63, 71]),                 # 1326 rows, 36 blocks: 54 tiles
    (64, 16, 512, [701, 1403, 2, 900, 1000, 37, 515, 8]),                          # 4558 rows, 96 blocks: 256 x 256 tiles, then the rest
    (128, 8, 512, [1402, 699, 3, 901, 1001, 38, 516, 5]),
    (64, 8, 1024, [130, 3, 257, 100]),                                        # 486 rows: split over K, a kernel of its own
])
@pytest.mark.parametrize("qk_norm", [False, True])
def test_cache_after_a_long_pass(hd, kv, H, lens, qk_norm):
    lens = np.array(lens, np.int32)
    shape = synth.ModelShape(1, H, kv, kv, hd, 64, 700, qk_norm=qk_norm)
    r = np.random.default_rng(hd + kv)
    blob, embed, cols = one_hot_keys_and_values(shape, r)
    ctx = make_ctx(shape, len(lens), int(lens.max()), blob)
    before = arena_now(ctx)
    toks = r.integers(0, shape.vocab, (len(lens), lens.max())).astype(np.int32)
    ctx.logprobs(toks, lens)
    check_cache(shape, ctx, before, toks, lens - 1, int(lens.max()), embed, cols)   # (the last token is only a target)
    ctx.close()


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("qk_norm", [False, True])
@pytest.mark.parametrize("rows", [256, 270, 600])   # 24 tiles: a kernel of its own; 48; 72
def test_rows_that_have_ended_append_nothing(hd, qk_norm, rows):
    """Decode steps whose rows are of sequences at positions of their own, and end one by one without being moved together."""
    shape, new = synth.ModelShape(1, 512, 8, 8, hd, 64, 700, qk_norm=qk_norm), 7
    if hd == 64:
        shape = shape.replace(n_q_heads=32)   # 96 weight blocks either way
    r = np.random.default_rng(hd + rows)
    blob, embed, cols = one_hot_keys_and_values(shape, r)
    ctx = make_ctx(shape, rows, 36 + new, blob)
    before = arena_now(ctx)
    lens = r.integers(1, 36, rows).astype(np.int32)
    prompts = r.integers(0, shape.vocab, (rows, 36)).astype(np.int32)
    stop = r.integers(1, new + 1, rows).astype(np.int32)
    stop[0] = new
    forced = r.integers(0, shape.vocab, (rows, new)).astype(np.int32)
    out = ctx.rollout(prompts, lens, 1, new, 1.0, 6, stop_lens=stop, forced=forced, no_compaction=True)
    assert np.array_equal(out["lens"], stop)
    strings = np.array([np.concatenate([prompts[n, :lens[n]], forced[n], prompts[n, lens[n]:]]) for n in range(rows)])
    check_cache(shape, ctx, before, strings, lens + stop - 1, 36 + new, embed, cols)
    ctx.close()


def test_which_launches_the_projection_takes(child):
    """Tiles too few to fill a fifth of the chip leave the post-processing to a kernel of its own."""
    child("""
s = synth.ModelShape(1, 512, 32, 8, 64, 64, 300)     # 96 weight blocks: 24 tiles per 256 rows

def launches(call):
    shim.hip_refuse(b"gemm_ring_qkv_kernel", 1 << 30)
    call()
    return shim.hip_seen()

ctx = make_ctx(s, 600, 600, synth.make_weights(s, 3))
p, l = synth.make_prompts(s.vocab, 1, 5, seed=2)
tokens = np.random.default_rng(5).integers(0, s.vocab, (1, 600)).astype(np.int32)
got = [launches(lambda: ctx.rollout(p, l, rows, 2, 1.0, 6)) for rows in (200, 256, 257, 600)]
got += [launches(lambda: ctx.logprobs(tokens, np.array([n + 1], np.int32))) for n in (200, 256, 257)]
want = [0, 0, 1, 1, 0, 0, 1]
print("as expected" if got == want else got)
""")
