"""The sampler fused into the lm_head against the fp32 sampler over the materialised logits of the same step: tokens must be the
same everywhere (both decide by the same fp32 scores; the logits are bit-identical), log-probs within fp32 rounding.
Vocabularies that end inside a weight block, inside a wavefront's share and on the first entry of a strip; every launch form by
batch size; temperatures at which the scores span thousands and at which they are nearly all noise."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("rows", [3, 100, 130])
@pytest.mark.parametrize("vocab", [32768, 32769, 163840, 163841])
def test_partials_of_a_row_at_the_edges_of_the_merge(rows, vocab):
    """A row's 256 partials of 128 entries, one for each thread of the merge, 1280, and one more than either; the logits of
    100 rows by workgroups of four blocks (32768) and of seven."""
    shape = synth.ModelShape(1, 64, 1, 1, 64, 64, vocab)
    ctx = make_ctx(shape, rows, 8, synth.make_weights(shape, 7))
    prompts, lens = synth.make_prompts(vocab, rows, 5, seed=2)
    forced = np.random.default_rng(rows).integers(0, vocab, size=(rows, 3)).astype(np.int32)
    a = ctx.rollout(prompts, lens, 1, 3, 1.0, 9, forced=forced)
    b = ctx.rollout(prompts, lens, 1, 3, 1.0, 9, forced=forced, unfused_sampler=True)
    assert np.array_equal(a["tokens"], b["tokens"])
    assert np.abs(a["logprobs"] - b["logprobs"]).max() < 2e-6 * max(8.0, np.abs(b["logprobs"]).max() + 0.1)   # as above
    ctx.close()


@pytest.mark.parametrize("vocab,dtype", [(1001, "fp32"), (4099, "bf16"), (9002, "fp32"), (9002, "bf16")])
def test_nucleus_draws_the_tokens_of_the_oracle_over_the_same_logits(orc, vocab, dtype):
    """Vocabularies whose rows are not aligned and end inside a group of four draws; a temperature at which nearly all mass is
    one token's, one at which the cut's bin holds a few keys and one at which every key shares a few bins (more of them than
    the candidate list holds)."""
    shape = synth.ModelShape(1, 256, 4, 2, 64, 512, vocab, dtype=dtype)
    blob = synth.make_weights(shape, 6)
    prompts, lens = synth.make_prompts(vocab, 3, 5, seed=vocab)
    ctx = make_ctx(shape, 3, 9, blob)
    forced = np.random.default_rng(vocab).integers(0, vocab, size=(3, 4)).astype(np.int32)
    checked = 0
    for temperature in (0.02, 1.0, 60.0):
        for top_p in (0.05, 0.95):
            got = ctx.rollout(prompts, lens, 1, 4, temperature, 17, top_p=top_p, forced=forced, want_logits=True)
            for n in range(3):
                for s in range(4):
                    z = got["logits"][n, s].astype(np.float64)
                    tok, lp, gap, kept, margin = orc.sample_top_p(z, temperature, top_p, 17, n, s)
                    # the kernel's masses carry the hardware exponential's error, relative 1e-6; its scores are fp32
                    size = max(8.0, np.abs(z).max() / temperature)
                    if margin < 4e-6 or gap < 1e-6 * size:
                        continue
                    checked += 1
                    assert got["tokens"][n, s] == tok, (temperature, top_p, n, s, kept)
                    assert abs(got["logprobs"][n, s] - lp) < 2e-6 * size, (temperature, top_p, n, s, kept)
    # of 72 draws; a row's 9002 masses are nearly equal at T = 60, so all rows' cuts lie as close to the 0.95 as the nearest
    # multiple of 1 / 9002 does (5e-6), and up to half a dozen of those 12 are left out
    assert checked >= 54
    ctx.close()


def _row(kind, vocab, r):
    z = r.standard_normal(vocab)
    if kind == "flat":
        z *= 1e-3
    elif kind == "spike over flat":      # half of the mass on one token, the cut among the others
        z *= 1e-4
        z[7] = np.log(vocab)
    elif kind == "a third equal":        # more equal logits than any list holds, in the middle of the others
        z[vocab // 3:2 * vocab // 3] = 0.25
    elif kind == "two values":
        z = np.where(z > 0, 1.0, 0.0)
    elif kind == "spike over equal":
        z[:] = 0.0
        z[vocab - 1] = np.log(vocab)
    return z


@pytest.mark.parametrize("kind", ["normal", "flat", "spike over flat", "a third equal", "two values", "spike over equal"])
@pytest.mark.parametrize("vocab", [1500, 32001, 151936])
def test_nucleus_of_rows_of_any_shape(orc, kind, vocab):
    """Rows whose scores spread over ten units, over a few thousandths, over thousandths below one large score, or fall on few
    values: the cut's bin then holds a few keys, has to be divided, or holds nothing but equal keys.  The model passes one vector
    on to the lm_head, whatever the token: 16 (1, 1/256, 0 ...), so two columns of lm_head are the row, in some 16 bits."""
    r = np.random.default_rng(vocab)
    shape = synth.ModelShape(1, 256, 4, 2, 64, 64, vocab)
    blob = synth.make_weights(shape, 1)
    off = synth.blob_offsets(shape)

    def tensor(name):
        at, dims = off[name]
        return blob[at:at + int(np.prod(dims))].view(*dims)
    for name in ("embed", "layers.0.wo", "layers.0.w_down", "lm_head"):
        tensor(name).zero_()
    tensor("embed")[:, 0], tensor("embed")[:, 1] = 1.0, 2.0 ** -8
    z = torch.from_numpy(_row(kind, vocab, r) / 16)
    head = tensor("lm_head")
    head[:, 0] = z
    head[:, 1] = (z - head[:, 0].double()) * 256
    ctx = make_ctx(shape, 2, 6, blob)
    prompts, lens = synth.make_prompts(vocab, 2, 3, seed=1)
    for top_p in (0.95, 0.6):
        got = ctx.rollout(prompts, lens, 1, 2, 1.0, 23, top_p=top_p, forced=np.zeros((2, 2), np.int32), want_logits=True)
        for n in range(2):
            for s in range(2):
                zz = got["logits"][n, s].astype(np.float64)
                tok, lp, gap, kept, _ = orc.sample_top_p(zz, 1.0, top_p, 23, n, s)
                # where the cut falls between nearly equal masses it may be one entry off: that entry's mass, 1 / (top_p vocab) at most
                # unless the spike is kept alone, goes to the log-sum-exp; its own draw is as unlikely as its mass
                assert gap < 1e-5 or got["tokens"][n, s] == tok, (top_p, n, s, kept)
                if got["tokens"][n, s] == tok:
                    assert abs(got["logprobs"][n, s] - lp) < 2.4e-5 + 2 / (top_p * kept), (top_p, n, s, kept)
    ctx.close()


@pytest.mark.parametrize("vocab", [1000, 9002])
def test_logits_of_nan_give_nan(vocab):
    """A snapshot with a NaN: the all-fp32 path, whose log-probs say so at every step, whether a row is sampled whole or in slices."""
    shape = synth.ModelShape(1, 256, 4, 2, 64, 512, vocab, dtype="fp32")
    blob = synth.make_weights(shape, 5).clone()
    at, _ = synth.blob_offsets(shape)["final_norm"]
    blob[at + 3] = float("nan")
    prompts, lens = synth.make_prompts(vocab, 3, 5, seed=1)
    ctx = make_ctx(shape, 3, 9, blob)
    for continuous in (False, True):
        got = ctx.rollout(prompts, lens, 1, 4, 1.0, 9, continuous=continuous)
        assert np.isnan(got["logprobs"]).all() and (got["lens"] == 4).all()
    ctx.close()
