"""The 16-bit attention kernel where its tiles, row groups and key ranges end, against the oracle: contexts around multiples
of a tile (32 keys) and of a workgroup's tiles (4 or 8 of them), rows around row tiles (16) and row groups (48), one tile per
wave and several, and rotary tables that do not start at a multiple of 16 bytes; the fp32 kernel where its ranges
grow past two tiles per wave."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev, host
from paper_2403_09919_amd import synth
from test_oracle_rope import tables

pytestmark = pytest.mark.gpu

# A probability is rounded to the storage type once and the result once; the values are averages of normal variates, |v| < 6
# (the bound the other attention tests use).
TOL = {"bf16": 2e-2, "f16": 4e-3}


@pytest.fixture(scope="module")
def rd():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2403_09919_amd import binding
    return binding


def _case(B, H, W, L, ctx, D, dtype, seed, vocab=32000):
    ctx = np.asarray(ctx, np.int32)
    N = W * L
    beams = synth.make_beams(B, W, L, vocab, seed, "uniform")
    q, kn, vn = synth.make_qkv_new(B, H, N, D, dtype, seed)
    kc, vc = synth.make_kv_cache(B, H, max(int(ctx.max()), 1), D, dtype, seed, ctx, True)
    return ctx, beams, q, kn, vn, kc, vc, oracle.dedup(beams, ctx)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("W,L", [(1, 1), (4, 4), (17, 1), (8, 5), (47, 1), (48, 1), (49, 1), (97, 1), (128, 3)])
@pytest.mark.parametrize("ctx", [(0, 1), (31, 33), (127, 129), (223, 256), (257, 700), (2048, 2049)])
def test_tile_and_group_edges(rd, dtype, D, W, L, ctx):
    announce(f"edges {dtype} D={D} W={W} L={L} ctx={ctx}")
    B, H = 2, 3
    ctx, beams, q, kn, vn, kc, vc, d = _case(B, H, W, L, ctx, D, dtype, W + L)
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], dtype, scale)
    dd = rd.rd_dedup(dev(beams), dev(ctx))
    out = rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), dd["n_packed"], dd["tree_mask_bits"], scale)
    torch.cuda.synchronize()
    got, want = synth.to_f64(host(out), dtype), synth.to_f64(ref, dtype)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL[dtype]
    for b in range(B):                                             # rows beyond the packed count are zero
        assert not got[b, :, int(d["n_packed"][b]):].any()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,L,ctx", [(8, 5, 300), (8, 5, 3000), (40, 4, 90)])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_rotary_tables_at_any_multiple_of_four_bytes(rd, D, W, L, ctx, shift):
    announce(f"rope tables D={D} W={W} L={L} ctx={ctx} shift={shift}")
    ctx, beams, q, kn, vn, kc, vc, d = _case(1, 2, W, L, [ctx], D, "bf16", D + W)
    scale, (cos, sin) = float(1.0 / np.sqrt(D)), tables(4096, D)
    dd = rd.rd_dedup(dev(beams), dev(ctx))

    def shifted(t):
        flat = torch.empty(t.size + 4, dtype=torch.float32, device="cuda")
        view = flat[shift:shift + t.size].view(t.shape)
        view.copy_(torch.from_numpy(t))
        return view

    def run(c, s):
        return rd.rd_tree_attn_rope(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), dd["n_packed"], dd["tree_mask_bits"],
                                    dd["position_ids"], c, s, scale)

    q2, k2 = dev(q), dev(kn)
    rd.rd_rope(q2, k2, dd["position_ids"], dd["n_packed"], dev(cos), dev(sin))
    sep = rd.rd_tree_attn(q2, dev(kc), dev(vc), dev(ctx), k2, dev(vn), dd["n_packed"], dd["tree_mask_bits"], scale)
    out, k_rot = run(shifted(cos), shifted(sin))
    torch.cuda.synchronize()
    P = int(d["n_packed"][0])
    assert np.array_equal(host(out), host(sep)) and np.array_equal(host(k_rot)[0, :, :P], host(k2)[0, :, :P])


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("H,W,L,ctx,vocabs", [(4, 70, 5, [1777], [1]), (4, 70, 5, [1777], [2]), (4, 70, 5, [4096], [3]), (3, 16, 5, [4096, 700, 3000], [2, 32000, 5]),
                                              (5, 30, 5, [2048, 2048], [2, 32000]), (2, 128, 3, [0, 3000, 31, 1500], [1, 4, 8, 32000]),
                                              (8, 50, 5, [3000, 2700], [2, 2]), (8, 50, 5, [3000, 2700], [2, 32000]), (3, 70, 5, [700, 650], [32000, 32000]),
                                              (4, 70, 5, [4000 - 37 * (7 * i % 20) for i in range(20)], [5] * 20)])
def test_few_packed_rows_in_a_wide_beam(rd, dtype, D, H, W, L, ctx, vocabs):
    """Candidates that share most of their prefixes (small vocabularies) beside ones that do not: the key ranges of a head go
    by how many of its row groups hold packed rows where all sequences agree in that (by the plan 8 and not 5 for 50 x 5 tokens, 4
    and not 7 for D=128, C=700, 2 and not 3 for the 20 sequences, longest first) and are the plan's usual ones where they differ."""
    announce(f"few packed rows {dtype} D={D} H={H} W={W} L={L} ctx={ctx} vocabs={vocabs}")
    B = len(ctx)
    ctx, _, q, kn, vn, kc, vc, _ = _case(B, H, W, L, ctx, D, dtype, W + H)
    beams = np.concatenate([synth.make_beams(1, W, L, v, 7 + i % 4, "uniform") for i, v in enumerate(vocabs)])
    d = oracle.dedup(beams, ctx)
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], dtype, scale)
    ws = rd.new_workspace(rd.rd_tree_attn_workspace(B, H, W * L, D, kc.shape[2], rd.RD_BF16 if dtype == "bf16" else rd.RD_F16), "cuda")
    for _ in range(2):                                             # the second call finds the counters as the first left them
        out = torch.full_like(dev(q), float("nan"))
        rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), dev(d["n_packed"]), dev(d["tree_mask_bits"]), scale,
                        out=out, workspace=ws)
        torch.cuda.synchronize()
        got, want = synth.to_f64(host(out), dtype), synth.to_f64(ref, dtype)
        assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL[dtype]
        for b in range(B):
            assert not got[b, :, int(d["n_packed"][b]):].any()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,L,C", [(3, 4, 60), (8, 5, 100), (8, 5, 190)])
def test_fp16_tiles_far_below_the_largest_score(rd, D, W, L, C):
    """One key draws nearly all of a row's weight and its value is zero (an attention sink), so the output is made of
    probabilities 2^-18.4 below it.  A tile's are taken against the tile's own maximum: relative to one reference for all tiles
    they would be subnormal in fp16, off by 2^-25 / 2^-18.4 = 1 %."""
    announce(f"sink D={D} W={W} L={L} C={C}")
    B, H, N = 1, 3, W * L
    ctx, beams, q, kn, vn, kc, vc, d = _case(B, H, W, L, [C], D, "f16", C)
    q[:], kn[:], kc[:] = 0, 0, 0
    q[..., 0], kc[:, :, 0, 0] = 1, 18.4 * np.log(2.0)               # the score of key 0; all others have none
    vc[:, :, :32] = 0
    vc[:, :, 32:C], vn[:] = np.abs(vc[:, :, 32:C]) + np.float16(0.5), np.abs(vn) + np.float16(0.5)
    npk, bits = dev(d["n_packed"]), dev(d["tree_mask_bits"])
    got = host(rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), npk, bits, 1.0))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], "f16", 1.0)
    P = int(d["n_packed"][0])
    sink = float(np.exp(np.float64(kc[0, 0, 0, 0])))
    mask = d["tree_mask"][0].astype(np.float64)[:P, :P]
    num = vc[0, :, 32:C].astype(np.float64).sum(1)[:, None] + np.einsum("pq,hqd->hpd", mask, vn[0, :, :P].astype(np.float64))
    want = num / (sink + (C - 1) + mask.sum(1))[None, :, None]
    # one rounding of the probabilities and one of the result to 11 bits, and the result lies among fp16's subnormals in part
    assert np.abs(ref[0, :, :P].astype(np.float64) - want).max() <= 2 ** -11 * want.max() + 2 ** -25
    assert (np.abs(got[0, :, :P].astype(np.float64) - want) <= 2 ** -10 * want + 2 ** -25).all()


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("W,L", [(3, 4), (8, 5), (12, 8)])
@pytest.mark.parametrize("C", [1, 40, 80, 100, 130, 165, 200, 230, 290, 560, 820, 1100, 1400, 1700, 2300])
def test_waves_without_a_tile_and_numbers_of_partials(rd, dtype, D, W, L, C):
    """One tile per wave at most: waves without one add nothing, whatever the launch before left in their LDS (here NaN), and
    heads of two to nine ranges are merged from as many partial results."""
    announce(f"idle waves {dtype} D={D} W={W} L={L} C={C}")
    H = 4
    ctx, beams, q, kn, vn, kc, vc, d = _case(1, H, W, L, [C], D, dtype, C + W)
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], dtype, scale)
    npk, bits = dev(d["n_packed"]), dev(d["tree_mask_bits"])
    nan = torch.full((1, H, 4000, D), float("nan"), dtype=dev(kc).dtype, device="cuda")
    rd.rd_tree_attn(dev(q), nan, nan, dev(np.array([4000], np.int32)), dev(kn), dev(vn), npk, bits, scale)
    out = rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), npk, bits, scale)
    torch.cuda.synchronize()
    got, want = synth.to_f64(host(out), dtype), synth.to_f64(ref, dtype)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL[dtype]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,L", [(1, 2), (4, 4), (8, 5), (20, 4)])
@pytest.mark.parametrize("ctx", [(0, 1), (15, 17), (111, 113), (127, 128), (225, 256), (370, 20), (604, 3), (1700, 900)])
def test_fp32_ranges_of_one_two_and_more_tiles_per_wave(rd, D, W, L, ctx):
    """Tiles of 16 keys, eight waves: waves of no, one, two and more tiles of a range.  Bound: the fp32 target."""
    announce(f"fp32 edges D={D} W={W} L={L} ctx={ctx}")
    ctx, beams, q, kn, vn, kc, vc, d = _case(2, 3, W, L, ctx, D, "f32", W + L)
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], "f32", scale)
    dd = rd.rd_dedup(dev(beams), dev(ctx))
    out = rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), dd["n_packed"], dd["tree_mask_bits"], scale)
    torch.cuda.synchronize()
    got = host(out)
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    for b in range(2):
        assert not got[b, :, int(d["n_packed"][b]):].any()


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("W,L,C", [(8, 5, 600), (8, 5, 1400), (12, 8, 700), (3, 2, 3000), (40, 5, 2000)])
def test_partials_of_several_xcds(rd, dtype, D, W, L, C):
    """Partial results from workgroups on different XCDs are read past the L2.  The runtime deals workgroups so that they do not
    occur; here the arrival words start with a square sum that no set of equal XCD numbers has.  A word is cleared by the call
    that merges, and where a head has one range it is not looked at."""
    announce(f"partials of several XCDs {dtype} D={D} W={W} L={L} C={C}")
    B, H = 1, 4
    ctx, beams, q, kn, vn, kc, vc, d = _case(B, H, W, L, [C], D, dtype, C + W)
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], dtype, scale)
    tq = dev(q)
    ws = rd.new_workspace(rd.rd_tree_attn_workspace(B, H, W * L, D, C, rd._dt_code(tq)), "cuda")
    n_rg = -(-W * L // (16 if dtype == "f32" else 48))
    ws[:8 * B * H * n_rg].view(torch.int64).fill_(1 << 32)
    out = rd.rd_tree_attn(tq, dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), dev(d["n_packed"]), dev(d["tree_mask_bits"]), scale, workspace=ws)
    torch.cuda.synchronize()
    got = synth.to_f64(host(out), dtype) if dtype != "f32" else host(out)
    want = synth.to_f64(ref, dtype) if dtype != "f32" else ref
    assert np.isfinite(got).all() and np.abs(got - want).max() <= (TOL[dtype] if dtype != "f32" else 1e-5 * np.abs(ref).max())
    words = ws[:8 * B * H * n_rg].view(torch.int64)
    assert ((words == 0) | (words == 1 << 32)).all() and (words == 0).any()      # merged heads' words; some head had partials
