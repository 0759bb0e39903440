"""SwiGLU where the gate's exponential leaves the range of fp32: gates of some hundreds, half of them negative, ups as much smaller, so that the
products are of ordinary size -- by the weight-streaming kernel (39 rows), the 256 x 128 ring tiles (512 rows) and the 256 x 256 ones (4096 rows), against
the fp64 oracle at every position of the first and the last string.

The scaled weights are exact: N(0, 0.02^2) times 2^10 stays below 255.9, where the packed halves (256 w) saturate, up to 12 standard deviations (2^12 would not:
3.1 of them, two weights in a thousand clipped and log-probs 1.1e-2 off).  Five values round to half on the way to a logit, by 2^-11 of themselves at most, and logits are N(0, 0.4^2): log-probs differ by
some 5 * 2^-11 * 0.4 * 4 standard deviations = 4e-3, inside BF16_LOGPROB_TOL; a NaN or a lost sign of one gate in a thousand does not pass."""
import numpy as np
import pytest

from oracle import oracle
from paper_2602_02192_amd import synth

from gpu_util import BF16_LOGPROB_TOL, make_ctx

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape(1, 384, 4, 2, 64, 1040, 500)   # gate/up: 65 weight blocks, nine strips of 256 columns


@pytest.mark.parametrize("n_seqs,length", [(1, 40), (2, 257), (16, 257)])
def test_gates_of_hundreds(n_seqs, length):
    blob = synth.make_weights(SHAPE, 4).clone()
    for name, by in (("w_gate", 2.0 ** 10), ("w_up", 2.0 ** -10)):
        at, dims = synth.blob_offsets(SHAPE)["layers.0." + name]
        blob[at:at + dims[0] * dims[1]] *= by
    toks = np.random.default_rng(n_seqs).integers(0, SHAPE.vocab, size=(n_seqs, length)).astype(np.int32)
    ctx = make_ctx(SHAPE, n_seqs, length, blob)
    got = ctx.logprobs(toks, np.full(n_seqs, length, np.int32), 1.0)
    ctx.close()
    orc, d, blob32 = oracle.load("f64"), oracle.desc_from_shape(SHAPE), synth.widen_to_f32(blob)
    for n in {0, n_seqs - 1}:
        ref = orc.logprobs(d, blob32, toks[n], 1.0)
        assert np.abs(got[n] - ref).max() < BF16_LOGPROB_TOL, n
