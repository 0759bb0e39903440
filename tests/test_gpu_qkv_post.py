"""What the QKV post kernels leave in the key cache, bit for bit: the narrow form (passes of fewer than 256 rows) and the wide
one.  The key and the value projection are the same one-hot rows, so the cached value is the key before norm and rotation, exact
in half precision, and the cached key has to be

    half(fma(a, cos, -fl(b sin))), half(fma(b, cos, fl(a sin)))

of its two halves a, b.  With a per-head norm (gains 1) the sum of squares runs over fma(b, b, fl(a a)) in the narrow form, over
fma(a, a, fl(b b)) in the wide one, as a tree over the dims; hd, eps and the gains leave its division and square root as the
only other roundings, both correctly rounded."""
import numpy as np
import pytest

from paper_2602_02192_amd import synth

from gpu_util import make_ctx

pytestmark = pytest.mark.gpu

F32, WIDE = np.float32, np.longdouble


def fma(a, b, c):   # products of halves and floats are exact in 64 bits of mantissa, and so, but for far-apart exponents, is the sum
    return (WIDE(a) * WIDE(b) + WIDE(c)).astype(F32)


def expected_keys(v, rope_base, norm_eps, wide):
    """v: float32 [heads, keys, hd], the keys before norm and rotation."""
    half = v.shape[-1] // 2
    a, b = v[..., :half], v[..., half:]
    if norm_eps is not None:
        t = fma(a, a, b * b) if wide else fma(b, b, a * a)
        lanes = np.arange(half)
        off = half // 2
        while off:
            t = t + t[..., lanes ^ off]
            off //= 2
        inv = F32(1) / np.sqrt(t / F32(2 * half) + F32(norm_eps))
        a, b = a * inv, b * inv
    ang = np.arange(v.shape[1])[:, None] * (float(rope_base) ** (-2.0 * np.arange(half) / (2 * half)))
    cos, sin = np.cos(ang).astype(F32), np.sin(ang).astype(F32)
    want = np.concatenate([fma(a, cos, -(b * sin)), fma(b, cos, a * sin)], -1)
    other = np.concatenate([fma(-b, sin, a * cos), fma(a, sin, b * cos)], -1)   # the other product rounded
    return want.astype(np.float16), other.astype(np.float16)


def tiles(cache, hd):
    """[heads, tiles, 64 * hd] halves -> keys and values [heads, keys, hd]."""
    h, t = cache.shape[:2]
    k = cache[:, :, :32 * hd].reshape(h, t, hd // 8, 32, 8).transpose(0, 1, 3, 2, 4).reshape(h, t * 32, hd)
    v = cache[:, :, 32 * hd:].reshape(h, t, 2, hd // 32, 2, 32, 8).transpose(0, 1, 2, 4, 6, 3, 5).reshape(h, t * 32, hd)
    return k, v


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("qk_norm", [False, True])
@pytest.mark.parametrize("n_seqs,length", [(1, 250), (5, 250)])   # 249 rows: narrow; 1245 rows: wide
def test_cached_keys_bit_for_bit(hd, qk_norm, n_seqs, length):
    kv, H = 8, 512
    shape = synth.ModelShape(1, H, kv, kv, hd, 64, 700, qk_norm=qk_norm)
    blob = synth.make_weights(shape, 3).clone()
    r = np.random.default_rng(5)
    at = 0
    for name, dims, _ in synth.tensor_table(shape):
        n = int(np.prod(dims))
        if name.endswith(("wk", "wv")):
            w = blob[at:at + n].view(*dims)
            w.zero_()
            cols = r.integers(0, H, dims[0]) if name.endswith("wk") else cols
            w[np.arange(dims[0]), cols] = 1.0
        at += n
    ctx = make_ctx(shape, n_seqs, length, blob)
    base = (-ctx.arena.data_ptr()) % 256
    before = ctx.arena[base:].clone()
    toks = r.integers(0, shape.vocab, (n_seqs, length)).astype(np.int32)
    ctx.logprobs(toks, np.full(n_seqs, length, np.int32))
    # the key cache is the first part of the arena, behind the weights, that a pass writes
    start = int((ctx.arena[base:] != before).nonzero()[0, 0]) // 256 * 256
    nt = (length + 31) // 32
    per_seq = kv * nt * 64 * hd
    raw = ctx.arena[base + start:base + start + n_seqs * per_seq * 2].cpu().numpy().view(np.float16).reshape(n_seqs, kv, nt, 64 * hd)
    differ = 0
    for n in range(n_seqs):
        k, v = tiles(raw[n], hd)
        k, v = k[:, :length - 1], v[:, :length - 1].astype(F32)
        assert np.abs(v).max() > 0.5
        want, other = expected_keys(v, shape.rope_base, shape.rms_eps if qk_norm else None, n_seqs > 1)
        assert np.array_equal(k, want), (n, int((k != want).sum()))
        differ += int((want != other).sum())
    assert differ > 0   # the rounding shows at these sizes
    ctx.close()
