"""rd_dedup, rd_accept and rd_accept_sample about 64 candidate tokens, up to which one wave holds a sequence: lanes without a token, masks
whose bits cross 32, candidates of one token and of 64, rows of one chunk and of several."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev, host, mask_bits_u64
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


@pytest.mark.parametrize("W,L", SHAPES)
def test_edges_of_a_wave_with_and_without_masks(rd, W, L):  # noqa: F811
    """The dense mask, the bit mask and prefix_tree are optional: every combination writes the rest, and nothing else."""
    announce("one wave, optional outputs W=%d L=%d" % (W, L))
    beams, ctx = synth.make_beams(3, W, L, 7, W + L, "high"), np.array([0, 9, 4000], np.int32)
    ref = oracle.dedup(beams, ctx)
    shapes = {k: ref[k].shape for k in ("prefix_tree", "packed_tokens", "n_packed", "unpack_index", "parent", "position_ids")}
    for dense, bits, prefix in itertools.product((False, True), repeat=3):
        out = {k: torch.full(s, -7, dtype=torch.int32, device="cuda") for k, s in shapes.items()}
        out["tree_mask"] = torch.full(ref["tree_mask"].shape, 9, dtype=torch.uint8, device="cuda") if dense else None
        out["tree_mask_bits"] = torch.full(ref["tree_mask_bits"].shape, -7, dtype=torch.int64, device="cuda") if bits else None
        if not prefix:
            out["prefix_tree"] = None
        rd.rd_dedup(dev(beams), dev(ctx), out=out)
        torch.cuda.synchronize()
        for k, v in out.items():
            if v is not None:
                assert np.array_equal(mask_bits_u64(v) if k == "tree_mask_bits" else host(v), ref[k]), (k, dense, bits, prefix)


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


@pytest.mark.parametrize("W,L", [(1, 2), (8, 8), (13, 5), (70, 5), (128, 3)])
@pytest.mark.parametrize("V", [900, 9000])
def test_sample_on_a_used_workspace(rd, W, L, V):  # noqa: F811
    """A call finds the arrival counters as the call before left them, cleared, and needs nothing of what else is in the workspace:
    here every other bit is set before a call.  Draws from the residual and from p, a first token refuted, several calls on one
    workspace, each as on a fresh one; after a call that draws from p alone the chunks' totals are as launch 1 cleared them."""
    announce("sample, used workspace W=%d L=%d V=%d" % (W, L, V))
    B, N = 3, W * L
    gen = torch.Generator(device="cuda").manual_seed(W + V)
    ws = rd.new_workspace(rd.rd_accept_sample_workspace(B, W, L, V), "cuda")
    totals = ws[256:256 + 4 * B * ((V + 4095) // 4096)]            # behind the counters
    for seed in range(4):
        ws[256:] = 255
        beams = synth.make_beams(B, W, L, V, seed, "uniform")
        d = rd.rd_dedup(dev(beams))
        logits = torch.randn((B, N, V), generator=gen, device="cuda") * 3
        draft = logits * (1 / 0.9) + (torch.randn((B, N, V), generator=gen, device="cuda") if seed % 2 else 0)      # (the same: all accepted)
        u, un = torch.rand((B, N), generator=gen, device="cuda") * 0.999, torch.rand((B,), generator=gen, device="cuda")
        root = dev(np.where(np.arange(B) == seed - 1, -1, beams[:, 0, 0]).astype(np.int32))
        got, want = (rd.rd_accept_sample(logits, draft, dev(beams), d["unpack_index"], d["n_packed"], u, un, 0.9, root_token=root, workspace=w)
                     for w in (ws, None))
        torch.cuda.synchronize()
        for k in want:
            assert torch.equal(got[k], want[k]), k
        assert not ws[:4 * B].any()
        if seed == 0:
            assert (got["best_len"] == L).all() and not totals.any()
        if seed == 3 and L > 2:
            assert (got["best_len"] < L).any()                     # (the residual is drawn from)
