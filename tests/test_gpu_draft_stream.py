"""The drafter's layers whose workgroups start apart in K, against the oracle: those of up to 8 rows (rd_stream_kernel) at the
edges of its tiles, one row to eight, rows of a sequence's own and of its candidates, columns that are no multiple of 16, shares of
K that differ by a unit between waves and the fewest units, one product and two; and those of more rows where K is a multiple of
2048 (rd_head_rows_kernel, rd_gemm_kernel), or their workgroups have half the columns; both weight layouts."""
import pytest
import torch

from draft_tolerance import inputs_small
from gpu_util import announce, dev
from test_gpu_draft import dev_params, rd, validate  # noqa: F401  (rd: the fixture)

pytestmark = pytest.mark.gpu

# The deviation of a plain fp32 evaluation from the oracle (draft_tolerance.fp32_deviation) is at most 3.7e-3 over these
# shapes, so the tolerance of test_gpu_draft (1e-2, derived from that deviation over its own shapes) covers them.
SHAPES = [(1024, 4099, 0, 1, 8, 3), (1024, 4111, 0, 8, 1, 3), (1088, 4001, 0, 2, 4, 3), (1536, 333, 1, 1, 5, 3), (1600, 96, 1, 7, 1, 3),
          (2112, 130, 1, 1, 8, 4), (2112, 130, 1, 3, 2, 3), (2176, 100, 0, 1, 1, 3),
          # 16, 40, 72 and 120 rows
          (1024, 16500, 0, 2, 8, 3), (1024, 16399, 0, 5, 8, 3), (2048, 130, 1, 5, 8, 3), (2048, 130, 1, 9, 8, 3), (1024, 16385, 1, 15, 8, 3),
          # up to 64 rows, 128 columns to a workgroup and K split: the last group whole, and half empty (the RNN's)
          (2624, 130, 1, 5, 8, 3), (2624, 130, 1, 8, 8, 2)]


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("Dm,V,K,B,W,L", SHAPES)
def test_layers_that_start_apart(rd, tiled, Dm, V, K, B, W, L):  # noqa: F811
    announce(f"draft stream Dm={Dm} V={V} K={K} B={B} W={W} L={L} tiled={tiled}")
    p, h, last = inputs_small(Dm, V, K, B, W, L)
    params = rd.rd_draft_pack(dev_params(p)) if tiled else dev_params(p)
    got = rd.rd_draft(params, dev(h), dev(last), W, L)
    torch.cuda.synchronize()
    validate(p, h, last, W, L, got, "draft")
