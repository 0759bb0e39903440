"""What the QKV projection of a long pass leaves in the cache when it rotates and appends in its own epilogue, bit for bit: both tile
forms, both head dims, head counts that no tile divides, sequences that start and end inside a block of 32 rows, sequences of one row,
a pass that goes on in the middle of a sequence.  The value projection repeats the key projection's one-hot rows, so cached
values are the keys before norm and rotation (exact in half precision), at the places that the cache's form gives them."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx
from test_gpu_qkv_post import F32, expected_keys, tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,kv,H,lens", [
    (64, 3, 512, [250, 2, 33, 260, 3, 9, 300, 257, 64, 65]),                       # 1243 rows, 18 weight blocks: 256 x 128 tiles
    (128, 3, 512, [251, 3, 2, 280, 34, 10, 299, 258, 66, 63]),                     # 36 blocks
    (64, 16, 512, [701, 1403, 2, 900, 1000, 37, 515, 8]),                          # 4558 rows, 96 blocks: 256 x 256 tiles, then the rest
    (128, 8, 512, [1402, 699, 3, 901, 1001, 38, 516, 5]),
    (64, 8, 1024, [130, 3, 257, 100]),                                        # 486 rows: split over K, a kernel of its own
])
@pytest.mark.parametrize("qk_norm", [False, True])
def test_cache_after_a_long_pass(hd, kv, H, lens, qk_norm):
    lens = np.array(lens, np.int32)
    shape = synth.ModelShape(1, H, kv, kv, hd, 64, 700, qk_norm=qk_norm)
    blob = synth.make_weights(shape, 3).clone()
    r = np.random.default_rng(hd + kv)
    at = 0
    for name, dims, _ in synth.tensor_table(shape):
        n = int(np.prod(dims))
        if name.endswith(("wk", "wv")):
            w = blob[at:at + n].view(*dims)
            w.zero_()
            cols = r.integers(0, H, dims[0]) if name.endswith("wk") else cols
            w[np.arange(dims[0]), cols] = 1.0
        elif name.endswith("embed"):
            embed = blob[at:at + n].view(*dims).float().numpy()
        at += n
    ctx = make_ctx(shape, len(lens), int(lens.max()), blob)
    base = (-ctx.arena.data_ptr()) % 256
    before = ctx.arena[base:].clone()
    toks = r.integers(0, shape.vocab, (len(lens), lens.max())).astype(np.int32)
    ctx.logprobs(toks, lens)
    start = int((ctx.arena[base:] != before).nonzero()[0, 0]) // 256 * 256
    nt = (int(lens.max()) + 31) // 32
    raw = ctx.arena[base + start:base + start + len(lens) * kv * nt * 64 * hd * 2].cpu().numpy().view(np.float16).reshape(len(lens), kv, nt, 64 * hd)
    for n, length in enumerate(lens):
        k, v = tiles(raw[n], hd)
        assert (k[:, length - 1:] == 0).all() and (v[:, length - 1:] == 0).all(), n   # nothing behind the last scored key
        k, v = k[:, :length - 1], v[:, :length - 1].astype(F32)
        # the values are the normed embedding at the one-hot columns, to within a rounding of half
        x = embed[toks[n, :length - 1]]
        x = (x / np.sqrt((x.astype(np.float64) ** 2).mean(-1, keepdims=True) + shape.rms_eps))[:, cols].reshape(length - 1, kv, hd).transpose(1, 0, 2)
        assert np.abs(v - x).max() <= 2.0 ** -10 * np.abs(x).max(), n
        want, _ = expected_keys(v, shape.rope_base, shape.rms_eps if qk_norm else None, True)
        assert np.array_equal(k, want), (n, int((k != want).sum()))
    ctx.close()
