"""The drafter's selection at the edges of its rules: candidates up to the most that are ranked by counting, lists up to one per
thread and past it, chunks with fewer tokens than candidates' groups, and vocabularies of equal logits."""
import numpy as np
import pytest

import torch

from draft_tolerance import inputs_small
from gpu_util import announce, dev, host
from paper_2403_09919_amd import synth
from test_gpu_draft import check, dev_params, rd  # noqa: F401  (rd: the fixture)
from test_oracle_draft import make_params

pytestmark = pytest.mark.gpu

# (Dm, V, K, B, W, L, tokens that share one row of the output layer).  Scores are compared with the tolerance of test_gpu_draft,
# whose derivation covers these models (hidden size 64, the same scale).
SHAPES = [(64, 300, 1, 2, 28, 3, 1), (64, 300, 1, 2, 29, 3, 1), (64, 5000, 1, 2, 28, 3, 1), (64, 4096, 1, 2, 1, 4, 1), (64, 4097, 1, 2, 5, 4, 1),
          (64, 33000, 1, 1, 16, 3, 1), (64, 33000, 1, 1, 17, 3, 1), (64, 70000, 0, 1, 8, 3, 1), (64, 20000, 1, 1, 28, 3, 1),
          (64, 9000, 1, 2, 17, 4, 3), (64, 9000, 1, 2, 10, 4, 64), (64, 9000, 1, 2, 9, 4, 700)]


def inputs(Dm, V, K, B, W, L, same):
    p, h, last = inputs_small(Dm, V, K, B, W, L)
    p["head_w"][:] = p["head_w"][np.arange(V) // same * same]
    return p, h, last


@pytest.mark.parametrize("Dm,V,K,B,W,L,same", SHAPES)
def test_selection_edges(rd, Dm, V, K, B, W, L, same):  # noqa: F811
    announce(f"draft selection Dm={Dm} V={V} K={K} B={B} W={W} L={L} same={same}")
    p, h, last = inputs(Dm, V, K, B, W, L, same)
    check(rd, p, h, last, W, L, "selection")
    if same > 1:                                            # equal logits: the smaller token first, so no gap below a chosen one
        beams = host(rd.rd_draft(dev_params(p), dev(h), dev(last), W, 2)["beams"])
        for b in range(B):
            chosen = set(beams[b, :, 1].tolist())
            for tok in chosen:
                assert all(x in chosen for x in range(tok // same * same, tok)), (b, tok)


@pytest.mark.parametrize("V,W", [(20000, 8), (20000, 28), (20000, 29), (40, 28), (140000, 4), (140000, 8)])
def test_equal_logits_take_the_smallest_tokens(rd, V, W):  # noqa: F811
    announce(f"draft selection, equal logits V={V} W={W}")
    p = make_params(V, 64, 0, 5)
    p["head_w"][:] = 0
    h = synth.f32_to_bf16_bits(np.ones((1, 64), np.float32))
    got = rd.rd_draft(dev_params(p), dev(h), dev(np.array([2], np.int32)), W, 4)
    torch.cuda.synchronize()
    assert host(got["beams"])[0].tolist() == [[2, 0, 0, w] for w in range(W)]
    assert np.allclose(host(got["beam_logp"]), -3 * np.log(V), atol=1e-4)


def test_nan_logits_keep_tokens_in_range(rd):  # noqa: F811
    announce("draft selection, NaN logits")
    V, W = 9000, 8
    p = make_params(V, 64, 1, 7)
    p["head_w"][5] = synth.f32_to_bf16_bits(np.full(128, np.nan, np.float32))
    h = synth.f32_to_bf16_bits(np.ones((1, 64), np.float32))
    got = rd.rd_draft(dev_params(p), dev(h), dev(np.array([2], np.int32)), W, 4)
    torch.cuda.synchronize()
    beams = host(got["beams"])
    assert (beams >= 0).all() and (beams < V).all()


@pytest.mark.parametrize("what", ["one logit +inf", "a chunk of -inf"])
@pytest.mark.parametrize("B,W,V", [(2, 1, 5000), (2, 4, 5000), (3, 12, 9000), (1, 28, 9000), (2, 3, 66000), (2, 20, 70000), (2, 40, 5000)])
def test_rows_without_a_score(rd, what, B, W, V):
    """A logit of +inf, or a whole chunk of 4096 logits at -inf, leaves a row without a finite log-sum-exp and all candidates
    without a score: the first candidate's largest logits are taken, whichever kernels run the selection."""
    announce(f"draft selection {what} B={B} W={W} V={V}")
    Dm, L = 128, 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W + V)

    def randn(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype).mul_(std)

    params = dict(emb=randn(V, Dm, std=0.8), rnn_u=randn(Dm, Dm, std=Dm ** -0.5), rnn_w=randn(Dm, Dm, std=Dm ** -0.5),
                  rnn_b=randn(Dm, std=0.01, dtype=torch.float32), mlp_w=randn(1, 2 * Dm, 2 * Dm, std=(2 * Dm) ** -0.5),
                  mlp_b=randn(1, 2 * Dm, std=0.01, dtype=torch.float32), head_w=randn(V, 2 * Dm, std=2 * (2 * Dm) ** -0.5))
    params["mlp_w"][0, Dm], params["mlp_b"][0, Dm] = 0, 50.0        # one input of the output layer is positive in every row
    if what == "one logit +inf":
        params["head_w"][77, Dm] = float("inf")
    else:
        params["head_w"][4096:8192, Dm] = float("-inf")
    last = torch.randint(0, V, (B,), generator=gen, device="cuda", dtype=torch.int32)
    r = rd.rd_draft(params, randn(B, Dm), last, W, L, steps=True)
    torch.cuda.synchronize()
    logits, beams = r["step_logits"].cpu(), r["beams"].cpu()
    assert (r["beam_logp"] == float("-inf")).all()
    for b in range(B):
        path = [int(last[b])]
        for t in range(L - 1):
            order = torch.argsort(logits[t, b * W], descending=True, stable=True)[:W].tolist()
            want = [path + [tok] for tok in order]
            path.append(order[0])
        assert beams[b].tolist() == want


@pytest.mark.parametrize("V,W", [(9000, 28), (9000, 5), (4996, 28), (4296, 28), (4100, 3), (20000, 16)])
@pytest.mark.parametrize("what", ["equal", "10 larger", "500 larger", "600 larger", "falling", "rising", "two values"])
def test_many_logits_at_the_bound(rd, what, V, W):  # noqa: F811
    """Vocabularies of few distinct logits: more of them than are kept reach the bound of a chunk's best."""
    announce(f"draft selection {what} V={V} W={W}")
    v = np.arange(V)
    rng = np.random.default_rng(V + W)
    z = {"equal": 0 * v, "10 larger": np.isin(v, rng.permutation(V)[:10]) * (v % 3 + 1), "500 larger": (v % 4096 < 500) * 1, "600 larger": (v % 4096 < 600) * 1,
         "falling": 255 - v % 4096 // 16, "rising": v % 4096 // 16, "two values": rng.integers(0, 2, V)}[what].astype(np.float32)
    p = make_params(V, 64, 0, 5)
    p["head_w"][:] = 0
    p["head_w"][:, 64] = synth.f32_to_bf16_bits(z)                  # logits z in every row (integers up to 255 are exact)
    h = synth.f32_to_bf16_bits(np.ones((2, 64), np.float32))
    got = rd.rd_draft(dev_params(p), dev(h), dev(np.array([2, 3], np.int32)), W, 2)
    torch.cuda.synchronize()
    order = np.argsort(-z, kind="stable")[:W]
    want = z[order].astype(np.float64) - np.log(np.exp((z - z.max()).astype(np.float64)).sum()) - z.max()
    for b, last in enumerate((2, 3)):
        assert host(got["beams"])[b].tolist() == [[last, int(t)] for t in order]
    assert np.allclose(host(got["beam_logp"]), want[None], atol=1e-4)
