"""rd_dedup and rd_accept about 64 candidate tokens, up to which one wave holds a sequence: lanes without a token, masks
whose bits cross 32, candidates of one token and of 64, rows of one chunk and of several."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev, host
from paper_2403_09919_amd import synth
from test_gpu_dedup_accept import check_accept, check_dedup, rd, run_accept  # noqa: F401  (rd: the fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 1), (1, 2), (1, 63), (1, 64), (1, 65), (64, 1), (63, 1), (65, 1), (32, 2), (2, 32), (31, 2), (2, 31), (33, 2),
          (16, 4), (4, 16), (8, 8), (21, 3), (3, 21), (13, 5), (5, 12), (5, 13), (12, 5), (6, 10)]


@pytest.mark.parametrize("W,L", SHAPES)
def test_edges_of_a_wave(rd, W, L):  # noqa: F811
    for seed, V, share in ((1, 2, "high"), (2, 7, "uniform"), (3, 4100, "high")):
        announce("one wave W=%d L=%d V=%d" % (W, L, V))
        beams = synth.make_beams(3, W, L, V, seed, share)
        check_dedup(rd, beams, np.array([0, 9, 4000], np.int32))
        d = oracle.dedup(beams)
        logits = synth.make_logits(3, W * L, V, seed, d["packed_tokens"], d["parent"], d["n_packed"], 0.9)
        for root in (None, beams[:, W - 1, 0].copy(), np.array([-1, beams[1, 0, 0], -1], np.int32)):
            check_accept(rd, logits, beams, root)


@pytest.mark.parametrize("W,L", [(4, 4), (16, 5)])
@pytest.mark.parametrize("V", [3, 900, 9000])
def test_rows_of_nan_end(rd, W, L, V):  # noqa: F811
    """Logits are NaN-free by contract; a row without any number has no arg max, and the call still ends."""
    announce("rows of NaN W=%d L=%d V=%d" % (W, L, V))
    beams = synth.make_beams(2, W, L, V, 5)
    d = oracle.dedup(beams)
    logits = synth.make_logits(2, W * L, V, 5, d["packed_tokens"], d["parent"], d["n_packed"], 0.9)
    want = oracle.argmax(logits, d["n_packed"])
    logits[1, 2, :] = np.nan
    want[1, 2] = -1
    assert np.array_equal(run_accept(rd, logits, beams, d, None)["argmax"], want)
