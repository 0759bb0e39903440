"""Scoring passes whose padded row count is 5, 6 or 7 blocks of 256 rows -- no multiple of the bands of four row blocks in which
the 256-row GEMM tiles are dealt to the XCDs, tile counts that are no multiple of eight, weight-block counts that no tile
divides -- against the fp64 oracle at every position."""
import numpy as np
import pytest

from oracle import oracle
from paper_2602_02192_amd import synth

from gpu_util import BF16_LOGPROB_TOL, make_ctx

pytestmark = pytest.mark.gpu

# gate/up: 172 weight blocks, 22 strips of 256 columns (132 and 154 tiles from six row blocks on; below that 256 x 128 tiles)
SHAPE = synth.ModelShape(1, 384, 8, 2, 64, 2752, 2100)


@pytest.mark.parametrize("n_seqs", [5, 6, 7])
def test_scoring_with_odd_row_block_counts(n_seqs):
    blob = synth.make_weights(SHAPE, 4, gain_jitter=0.1)
    blob32 = synth.widen_to_f32(blob)
    rng = np.random.default_rng(n_seqs)
    toks = rng.integers(0, SHAPE.vocab, size=(n_seqs, 257)).astype(np.int32)   # 256 scored rows each
    lens = np.full(n_seqs, 257, np.int32)
    lens[1] = 200                                                              # rows of a block from two sequences
    ctx = make_ctx(SHAPE, n_seqs, 257, blob)
    got = ctx.logprobs(toks, lens, 1.0)
    orc, d = oracle.load("f64"), oracle.desc_from_shape(SHAPE)
    for n in range(n_seqs):
        ref = orc.logprobs(d, blob32, toks[n, :lens[n]], 1.0)
        assert np.abs(got[n, :lens[n]] - ref).max() < BF16_LOGPROB_TOL, n
        assert (got[n, lens[n]:] == 0).all()
    ctx.close()
