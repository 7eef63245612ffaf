"""rd_dedup beyond 64 candidate tokens, whole candidates to a wave, bit for bit against the oracle: candidates that fill a wave's
lanes or leave some, a last wave that is not full, most waves, candidates of 64 tokens and of 65 (the other kernel), token counts
that are odd, even and multiples of 4 (the dense mask is written in three ways), the last rows of the mask; every combination of
the optional outputs."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev, host, mask_bits_u64
from paper_2403_09919_amd import synth
from test_gpu_dedup_accept import check_dedup, rd  # noqa: F401  (rd: the fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(13, 5), (14, 5), (33, 2), (128, 3), (127, 3), (100, 1), (11, 33), (12, 32), (17, 22), (6, 64), (5, 65), (2, 64), (2, 33), (7, 11),
          (9, 15), (25, 6), (16, 16), (24, 16), (70, 5), (3, 127)]


@pytest.mark.parametrize("W,L", SHAPES)
def test_candidates_by_waves(rd, W, L):  # noqa: F811
    announce("dedup waves W=%d L=%d" % (W, L))
    for seed, V, share in ((1, 1, "high"), (2, 2, "high"), (3, 3, "uniform"), (4, 32000, "high")):
        check_dedup(rd, synth.make_beams(3, W, L, V, seed, share), np.array([0, 9, 4000], np.int32))
    beams, ctx = synth.make_beams(3, W, L, 7, W + L, "high"), np.array([0, 9, 4000], np.int32)
    ref = oracle.dedup(beams, ctx)
    names = ("prefix_tree", "packed_tokens", "n_packed", "unpack_index", "parent", "position_ids")
    for dense, bits, prefix in itertools.product((False, True), repeat=3):
        out = {k: torch.full(ref[k].shape, -7, dtype=torch.int32, device="cuda") for k in names}
        out["tree_mask"] = torch.full(ref["tree_mask"].shape, 9, dtype=torch.uint8, device="cuda") if dense else None
        out["tree_mask_bits"] = torch.full(ref["tree_mask_bits"].shape, -7, dtype=torch.int64, device="cuda") if bits else None
        if not prefix:
            out["prefix_tree"] = None
        rd.rd_dedup(dev(beams), dev(ctx), out=out)
        torch.cuda.synchronize()
        for k, v in out.items():
            if v is not None:
                assert np.array_equal(mask_bits_u64(v) if k == "tree_mask_bits" else host(v), ref[k]), (k, dense, bits, prefix)
