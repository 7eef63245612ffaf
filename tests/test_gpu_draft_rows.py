"""The drafter's layers of many rows (rd_gemm_kernel) at the edges of its tiles, against the oracle: rows around 32, 64,
128 and 256 (its row tiles, and the launches a call is cut into), columns that are no multiple of 16 or of the 256 of a
workgroup, more column groups than workgroups of a launch (K not split), and the smallest K, both weight layouts."""
import pytest
import torch

from draft_tolerance import inputs_small
from gpu_util import announce, dev
from test_gpu_draft import dev_params, rd, validate  # noqa: F401  (rd: the fixture)

pytestmark = pytest.mark.gpu

# The deviation of a plain fp32 evaluation from the oracle (draft_tolerance.fp32_deviation) is at most 8.1e-4 over these
# shapes, so the tolerance of test_gpu_draft (1e-2, derived from that deviation over its own shapes) covers them.
SHAPES = [(64, 130, 1, 11, 3, 3), (64, 257, 2, 8, 8, 3), (192, 1000, 2, 5, 13, 3), (64, 301, 1, 16, 8, 3), (128, 515, 2, 43, 3, 3),
          (320, 777, 1, 32, 8, 4), (64, 300, 1, 257, 1, 3), (64, 400, 2, 6, 50, 3), (64, 333, 0, 128, 4, 3), (64, 70003, 1, 13, 10, 3),
          # 64 rows and fewer: layers too large for the unsplit kernel, K split, not split and in workgroups of 128 columns
          (320, 14000, 0, 5, 8, 3), (64, 66000, 0, 6, 10, 3), (192, 24000, 0, 5, 8, 3), (192, 24000, 0, 10, 8, 3),
          # 9 to 32 rows of layers large enough for it, both products of the RNN too
          (2944, 200, 1, 4, 4, 2), (2944, 100, 1, 17, 1, 2), (5056, 100, 1, 9, 1, 2), (4160, 100, 0, 8, 2, 3), (4096, 100, 0, 1, 32, 3),
          (6144, 64, 1, 11, 1, 2), (6144, 64, 1, 10, 1, 2)]


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("Dm,V,K,B,W,L", SHAPES)
def test_rows_and_columns_at_the_edges(rd, tiled, Dm, V, K, B, W, L):  # noqa: F811
    announce(f"draft rows Dm={Dm} V={V} K={K} B={B} W={W} L={L} tiled={tiled}")
    p, h, last = inputs_small(Dm, V, K, B, W, L)
    params = rd.rd_draft_pack(dev_params(p)) if tiled else dev_params(p)
    got = rd.rd_draft(params, dev(h), dev(last), W, L)
    torch.cuda.synchronize()
    validate(p, h, last, W, L, got, "draft")
