"""The drafter's layers of 33 to 128 rows in workgroups of 13 to 15 column tiles (rd_gemm_kernel where 16 leave compute units
without one), K split and not, both row-tile instances and both weight layouts, against the oracle.  The output layer's K is no
multiple of 256, so that this kernel runs it."""
import pytest
import torch

from draft_tolerance import inputs_small
from gpu_util import announce, dev
from test_gpu_draft import dev_params, rd, validate  # noqa: F401  (rd: the fixture)

pytestmark = pytest.mark.gpu

# Columns: 24001 are 94 groups of 16 tiles or 116 of 13, in two splits; 27000 are 121 of 14; 40001 are 193 of 13, K not split, an odd
# number of rounds of two k-steps where K is 2176.  The deviation of a plain fp32 evaluation from the oracle
# (draft_tolerance.fp32_deviation) is at most 2e-4 over them, so the tolerance of test_gpu_draft covers them.
SHAPES = [(2112, 24001, 0, 40, 1, 2), (2112, 24001, 0, 72, 1, 2), (2112, 27000, 0, 70, 1, 2), (1088, 40001, 0, 35, 1, 3),
          (1088, 40001, 0, 12, 8, 3)]


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("Dm,V,K,B,W,L", SHAPES)
def test_fewer_columns_per_workgroup(rd, tiled, Dm, V, K, B, W, L):  # noqa: F811
    announce(f"draft columns Dm={Dm} V={V} K={K} B={B} W={W} L={L} tiled={tiled}")
    p, h, last = inputs_small(Dm, V, K, B, W, L)
    params = rd.rd_draft_pack(dev_params(p)) if tiled else dev_params(p)
    got = rd.rd_draft(params, dev(h), dev(last), W, L)
    torch.cuda.synchronize()
    validate(p, h, last, W, L, got, "draft")
