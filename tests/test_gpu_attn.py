"""GPU parity, tree attention: rd_tree_attn against the CPU oracle.

Tolerances (stated by the benchmark spec, written here): fp32 -> max|gpu-ref| <= 1e-5 * max|ref| over
the tensor; bf16 -> max|gpu-ref| <= 2e-2."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import announce, dev, host
from paper_2403_09919_amd import synth

pytestmark = pytest.mark.gpu

F32_REL = 1e-5
BF16_ABS = 2e-2
F16_ABS = 5e-3       # fp16: probabilities and output carry 11 significand bits (2^-11 relative each)


@pytest.fixture(scope="module")
def rd():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2403_09919_amd import binding
    return binding


def gpu_attn(rd, t, d, dtype, scale, workspace=None):
    out = rd.rd_tree_attn(dev(t["q"]), dev(t["k_cache"]), dev(t["v_cache"]), dev(t["ctx_len"]),
                          dev(t["k_new"]), dev(t["v_new"]), dev(d["n_packed"]), dev(d["tree_mask_bits"]),
                          scale, workspace=workspace)
    torch.cuda.synchronize()
    return host(out)


def compare(got, ref, dtype, what=""):
    g, r = synth.to_f64(got, dtype), synth.to_f64(ref, dtype)
    assert np.isfinite(g).all(), "non-finite output " + what
    err = np.abs(g - r).max()
    if dtype == "f32":
        assert err <= F32_REL * max(np.abs(r).max(), 1e-30), (what, err, np.abs(r).max())
    else:
        assert err <= (F16_ABS if dtype == "f16" else BF16_ABS), (what, err)
    return err


def n_row_groups(N):
    """Row groups (each of at most three 16-row tiles) of a head in the 16-bit kernel: an arrival word of 8 bytes each."""
    tiles = -(-N // 16)
    per = -(-tiles // -(-tiles // 3))
    return -(-tiles // per)


def make_case(B, H, D, W, L, ctx, dtype, seed, V=6, share="uniform", poison=True):
    ctx = np.asarray(ctx, np.int32)
    Cmax = int(max(ctx.max(), 0))
    t = dict(ctx_len=ctx, beams=synth.make_beams(B, W, L, V, seed, share))
    t["q"], t["k_new"], t["v_new"] = synth.make_qkv_new(B, H, W * L, D, dtype, seed)
    t["k_cache"], t["v_cache"] = synth.make_kv_cache(B, H, Cmax, D, dtype, seed, ctx, poison)
    return t


def full_check(rd, t, dtype, scale=None, what=""):
    B, H, N, D = t["q"].shape
    scale = float(1.0 / np.sqrt(D)) if scale is None else scale
    d = oracle.dedup(t["beams"], t["ctx_len"])
    ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                           d["n_packed"], d["tree_mask"], dtype, scale)
    got = gpu_attn(rd, t, d, dtype, scale)
    for b in range(B):                                   # rows beyond the packed count are exactly zero
        assert (synth.to_f64(got, dtype)[b, :, int(d["n_packed"][b]):] == 0).all()
    return compare(got, ref, dtype, what)


def test_config1_tiny_fp32(rd):
    cfg = synth.CONFIGS[1]
    announce("attn config 1 (fp32)")
    t = synth.make_attn_inputs(cfg)
    full_check(rd, t, "f32", what="cfg1")


def test_config2_vicuna7b_full(rd):
    cfg = synth.CONFIGS[2]
    announce("attn config 2 (bf16, whole tensor)")
    t = synth.make_attn_inputs(cfg)
    err = full_check(rd, t, "bf16", what="cfg2")
    print("cfg2 max abs err", err)


@pytest.mark.parametrize("idx", [3, 4, 5])
def test_full_size_configs_whole_tensor(rd, idx):
    """Full-size tensors in the launches the benchmark uses (four-wave workgroups with three row tiles; config 3: one key range
    per head; config 4: two row groups of one range each; config 5: two row groups, longest sequences first), every head and every
    row against the oracle."""
    cfg = synth.CONFIGS[idx]
    announce("attn config %d (bf16, full size, whole tensor)" % idx)
    t = synth.make_attn_inputs(cfg)
    err = full_check(rd, t, cfg.dtype, what="cfg%d" % idx)
    print("cfg%d whole-tensor max abs err %.3e" % (idx, err))


def test_four_wave_three_tiles_whole_tensor(rd):
    """More heads than compute units and more than 64 MB of K/V: four-wave workgroups with three row tiles, one key range per head, ragged contexts; every
    head and row against the oracle."""
    announce("attn bf16, 320 heads, 4-wave workgroups, whole tensor")
    B, H, D, W, L = 10, 32, 128, 8, 5
    ctx = [704, 641, 577, 700, 513, 690, 1, 333, 704, 129]
    assert 2 * B * H * max(ctx) * D * 2 >= 64e6 and B * H > 256
    t = make_case(B, H, D, W, L, ctx, "bf16", seed=320, V=32000)
    full_check(rd, t, "bf16", what="4-wave-3-tiles")


def test_fp16_large_cache_whole_tensor(rd):
    """IEEE-half K/V of more than 64 MB: four-wave workgroups, three key ranges."""
    announce("attn fp16, 67 MB of K/V, whole tensor")
    B, H, D, W, L, C = 2, 32, 128, 8, 5, 2048
    assert 2 * B * H * C * D * 2 >= 64e6
    t = make_case(B, H, D, W, L, [C, C - 37], "f16", seed=64, V=32000)
    full_check(rd, t, "f16", what="f16-large")


def test_full_size_configs_sampled_rows_unrounded(rd):
    """Config 5 once more on sampled rows against the oracle's unrounded (fp64) rows: bounds the
    kernel's own error without the reference's final rounding."""
    cfg = synth.CONFIGS[5]
    announce("attn config 5 (bf16, full size, sampled unrounded rows)")
    t = synth.make_attn_inputs(cfg)
    d = oracle.dedup(t["beams"], t["ctx_len"])
    scale = float(1.0 / np.sqrt(cfg.D))
    got = synth.to_f64(gpu_attn(rd, t, d, cfg.dtype, scale), cfg.dtype)
    rng = np.random.default_rng(5)
    rows = []
    for b in range(cfg.B):
        P = int(d["n_packed"][b])
        for h in rng.choice(cfg.H, size=3, replace=False):
            for p in sorted(set([0, P - 1] + rng.integers(0, P, size=3).tolist())):
                rows.append((b, int(h), int(p)))
    ref = oracle.tree_attn_rows(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                                d["n_packed"], d["tree_mask"], cfg.dtype, scale, rows)
    err = max(np.abs(got[b, h, p] - ref[n]).max() for n, (b, h, p) in enumerate(rows))
    assert err <= BF16_ABS


@pytest.mark.parametrize("dtype", ["bf16", "f32", "f16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,L", [(1, 1), (1, 5), (3, 5), (4, 4), (7, 5), (8, 8), (13, 6), (16, 6), (16, 7), (64, 2), (1, 128)])
def test_shapes(rd, dtype, D, W, L):
    """Every packed-row tile count (N = 1 .. 128), both head sizes, ragged contexts that end
    inside a tile, inside a block, at zero, and beyond several blocks."""
    announce("attn shapes dtype=%s D=%d W=%d L=%d" % (dtype, D, W, L))
    ctx = [0, 1, 31, 129, 300, 517]
    t = make_case(len(ctx), 2, D, W, L, ctx, dtype, seed=W * 131 + L)
    full_check(rd, t, dtype, what="shapes")


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,H,W,L,ctx", [(2, 8, 3, 4, (700, 1100)), (1, 3, 8, 5, (1500,)), (3, 2, 12, 6, (40, 513, 900)), (1, 2, 40, 6, (800,))])
def test_scores_that_rise(rd, dtype, D, B, H, W, L, ctx):
    """Softmax references that move block after block: keys that grow along the context (and, in the second half of
    the heads, a few late keys far above the rest), so that earlier blocks' sums are rescaled, for some rows only."""
    announce("attn rising scores dtype=%s D=%d B=%d H=%d W=%d L=%d" % (dtype, D, B, H, W, L))
    t = make_case(B, H, D, W, L, ctx, dtype, seed=D + W, poison=False)
    Cmax = max(ctx)
    k = synth.to_f64(t["k_cache"], dtype)
    rise = np.linspace(0.05, 4.0, Cmax)[None, None, :, None]
    k[:, :H // 2 + 1] *= rise
    k[:, H // 2 + 1:, ::97] *= 6.0
    if dtype == "bf16":
        t["k_cache"] = host(torch.from_numpy(k).to(torch.bfloat16))
    else:
        t["k_cache"] = k.astype(np.float16 if dtype == "f16" else np.float32)
    full_check(rd, t, dtype, scale=0.5, what="rising")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D,B,H,W,L,Cmax", [(128, 3, 3, 8, 5, 4000), (64, 2, 5, 3, 4, 6000), (128, 1, 2, 30, 6, 3000), (128, 1, 9, 70, 5, 2500)])
def test_live_contexts_far_below_capacity(rd, dtype, D, B, H, W, L, Cmax):
    """Plans with many workgroups per head, contexts that leave most of them without keys, head counts that do not
    divide by the XCDs."""
    announce("attn far below capacity dtype=%s D=%d B=%d H=%d W=%d L=%d" % (dtype, D, B, H, W, L))
    for ctx in ([0, 33, 250][:B], [Cmax, 31, 700][:B]):
        ctx = np.asarray(ctx, np.int32)
        t = dict(ctx_len=ctx, beams=synth.make_beams(B, W, L, 9, 3, "uniform"))
        t["q"], t["k_new"], t["v_new"] = synth.make_qkv_new(B, H, W * L, D, dtype, 4)
        t["k_cache"], t["v_cache"] = synth.make_kv_cache(B, H, Cmax, D, dtype, 5, ctx, True)
        full_check(rd, t, dtype, what="below capacity")


@pytest.mark.parametrize("dtype", ["bf16", "f32", "f16"])
def test_degenerate_beams_and_scales(rd, dtype):
    announce("attn degenerate beams dtype=%s" % dtype)
    B, H, D, W, L = 2, 3, 128, 8, 5
    t = make_case(B, H, D, W, L, [200, 77], dtype, seed=5)
    t["beams"][:] = np.array([4, 3, 2, 1, 0], np.int32)           # all identical -> P = L
    full_check(rd, t, dtype, what="identical")
    t["beams"] = np.arange(B * W * L, dtype=np.int32).reshape(B, W, L)   # all distinct -> P = W*L
    full_check(rd, t, dtype, what="distinct")
    full_check(rd, t, dtype, scale=0.0, what="scale0")            # uniform average of visible values
    full_check(rd, t, dtype, scale=1.0, what="scale1")            # peaked softmax


@pytest.mark.parametrize("dtype", ["bf16", "f32", "f16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,L,V", [(70, 5, 6), (64, 6, 3), (1, 384, 5), (128, 3, 2), (29, 5, 50), (20, 7, 4), (50, 5, 1000)])
def test_wide_beams(rd, dtype, D, W, L, V):
    """The paper's widest beams (Sec. 4.3: up to 70 candidates of 5 tokens) and beyond: packed rows
    in several row groups, packed keys in several blocks, mask rows of up to six words."""
    announce("attn wide beams dtype=%s D=%d W=%d L=%d V=%d" % (dtype, D, W, L, V))
    ctx = [0, 97, 700]
    t = make_case(len(ctx), 2, D, W, L, ctx, dtype, seed=W * 7 + L, V=V)
    full_check(rd, t, dtype, what="wide")


def test_wide_beams_config2_shape(rd):
    announce("attn wide beams, Vicuna-7B-shaped layer with 70 candidates")
    t = make_case(1, 32, 128, 70, 5, [1024], "bf16", seed=70, V=32000, share="high")
    full_check(rd, t, "bf16", what="wide-7b")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_many_splits_long_context(rd, dtype):
    announce("attn long ragged context, many splits, " + dtype)
    t = make_case(2, 4, 128, 8, 5, [5000, 2311], dtype, seed=21, V=3)
    full_check(rd, t, dtype, what="long")


def test_config2_shape_fp16(rd):
    """The Vicuna-7B-shaped layer with half-precision K/V (App. A.2 runs its drafting in float16)."""
    announce("attn config 2 shape, fp16")
    cfg = synth.CONFIGS[2]
    t = make_case(cfg.B, cfg.H, cfg.D, cfg.W, cfg.L, [cfg.ctx_hi], "f16", seed=cfg.seed, V=cfg.V)
    full_check(rd, t, "f16", what="cfg2-f16")


def test_workspace_reuse_and_determinism(rd):
    announce("attn workspace reuse, run-twice determinism")
    t = make_case(2, 8, 128, 8, 5, [700, 1024], "bf16", seed=3)
    d = oracle.dedup(t["beams"], t["ctx_len"])
    nbytes = rd.rd_tree_attn_workspace(2, 8, 40, 128, 1024, rd.RD_BF16)
    ws = rd.new_workspace(nbytes, "cuda")
    a = gpu_attn(rd, t, d, "bf16", 0.1, ws)
    b = gpu_attn(rd, t, d, "bf16", 0.1, ws)
    assert np.array_equal(a, b)
    nctr = 2 * 8                                           # one 8-byte arrival word per (sequence, head)
    assert int(ws[: 8 * nctr].to(torch.int64).sum()) == 0
    ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                           d["n_packed"], d["tree_mask"], "bf16", 0.1)
    compare(a, ref, "bf16")


@pytest.mark.parametrize("shape", ["config2", "row-groups"])
def test_workspace_reused_by_different_inputs_back_to_back(rd, shape):
    """Eight DIFFERENT inputs of one shape go through ONE workspace back to back, with no
    synchronisation in between, each into its own output; every output is compared with the oracle.
    A merge that read a partial result or an arrival word left by the previous call would show here.
    Shapes: the Vicuna-7B-shaped layer (five ranges of the context's and the packed keys per head) and a long
    context whose heads have two row groups of seven ranges."""
    if shape == "config2":
        B, H, D, W, L, ctxs = 1, 32, 128, 8, 5, [[1024]] * 8
    else:
        B, H, D, W, L = 2, 8, 128, 16, 5
        ctxs = [[4096, 4096 - 301 * i] for i in range(8)]
    Cmax = 4096 if shape != "config2" else 1024
    N = W * L
    announce("attn stale-workspace check, %s, 8 inputs through one workspace" % shape)
    ws = rd.new_workspace(rd.rd_tree_attn_workspace(B, H, N, D, Cmax, rd.RD_BF16), "cuda")
    scale = float(1.0 / np.sqrt(D))
    cases, outs = [], []
    for i in range(8):
        t = make_case(B, H, D, W, L, ctxs[i], "bf16", seed=1000 + 17 * i, V=32000, poison=False)
        if t["k_cache"].shape[2] < Cmax:                   # every call uses the same Cmax (one workspace layout)
            pad = Cmax - t["k_cache"].shape[2]
            t["k_cache"] = np.pad(t["k_cache"], ((0, 0), (0, 0), (0, pad), (0, 0)))
            t["v_cache"] = np.pad(t["v_cache"], ((0, 0), (0, 0), (0, pad), (0, 0)))
        d = oracle.dedup(t["beams"], t["ctx_len"])
        td = {k: dev(v) for k, v in t.items()}
        td["n_packed"], td["mask"] = dev(d["n_packed"]), dev(d["tree_mask_bits"])
        cases.append((t, d, td))
    torch.cuda.synchronize()
    for t, d, td in cases:                                 # back to back on one stream, no sync
        outs.append(rd.rd_tree_attn(td["q"], td["k_cache"], td["v_cache"], td["ctx_len"], td["k_new"], td["v_new"],
                                    td["n_packed"], td["mask"], scale, workspace=ws))
    torch.cuda.synchronize()
    for i, ((t, d, td), o) in enumerate(zip(cases, outs)):
        ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                               d["n_packed"], d["tree_mask"], "bf16", scale)
        compare(host(o), ref, "bf16", "reuse %s #%d" % (shape, i))
    words = 8 * B * H * n_row_groups(N)
    assert ws.numel() > 2 * words and int(ws[:words].to(torch.int64).sum()) == 0       # arrival words are left clear


def test_whole_path_chained_on_device(rd):
    """rd_dedup -> rd_tree_attn -> rd_accept with device-resident intermediates equals the oracle chain."""
    cfg = synth.CONFIGS[2]
    announce("whole path, config 2")
    t = synth.make_attn_inputs(cfg)
    scale = float(1.0 / np.sqrt(cfg.D))
    dref = oracle.dedup(t["beams"], t["ctx_len"])
    logits = synth.make_logits(cfg.B, cfg.N, cfg.V, cfg.seed, dref["packed_tokens"], dref["parent"],
                               dref["n_packed"], cfg.p_plant)
    ref = oracle.verify_step(t["beams"], t["ctx_len"], t["q"], t["k_cache"], t["v_cache"], t["k_new"],
                             t["v_new"], logits, cfg.dtype, scale)
    beams_d, ctx_d = dev(t["beams"]), dev(t["ctx_len"])
    dd = rd.rd_dedup(beams_d, ctx_d)
    out = rd.rd_tree_attn(dev(t["q"]), dev(t["k_cache"]), dev(t["v_cache"]), ctx_d, dev(t["k_new"]),
                          dev(t["v_new"]), dd["n_packed"], dd["tree_mask_bits"], scale)
    acc = rd.rd_accept(dev(logits), beams_d, dd["unpack_index"], dd["n_packed"])
    torch.cuda.synchronize()
    for k in ("packed_tokens", "n_packed", "unpack_index", "parent", "position_ids", "tree_mask"):
        assert np.array_equal(host(dd[k]), ref[k]), k
    compare(host(out), ref["attn_out"], cfg.dtype, "chain")
    assert np.array_equal(host(acc["argmax"]), ref["argmax"])
    for k in ("n_accept", "best_beam", "best_len", "next_token", "accepted_idx"):
        assert np.array_equal(host(acc[k]), ref[k]), k


def test_graph_replay_matches_eager(rd):
    """The library only enqueues kernels, so a caller may capture a step into a HIP graph.
    Replays (with eager work and synchronisations in between) must reproduce the eager result."""
    announce("whole path captured in a HIP graph, 3 replays")
    t = make_case(2, 4, 128, 8, 5, [300, 1000], "bf16", seed=17, poison=False)
    B, W, L, H, D, N, V = 2, 8, 5, 4, 128, 40, 2000
    dref = oracle.dedup(t["beams"], t["ctx_len"])
    logits = synth.make_logits(B, N, V, 17, dref["packed_tokens"], dref["parent"], dref["n_packed"], 0.7)
    td = {k: dev(v) for k, v in t.items()}
    lg = dev(logits)
    ws_a = rd.new_workspace(rd.rd_tree_attn_workspace(B, H, N, D, 1000, rd.RD_BF16), "cuda")
    ws_c = rd.new_workspace(rd.rd_accept_workspace(B, W, L, V), "cuda")
    state = {}

    def step():
        state["d"] = rd.rd_dedup(td["beams"], td["ctx_len"], out=state.get("d"))
        d = state["d"]
        state["o"] = rd.rd_tree_attn(td["q"], td["k_cache"], td["v_cache"], td["ctx_len"], td["k_new"], td["v_new"],
                                     d["n_packed"], d["tree_mask_bits"], 0.09, out=state.get("o"), workspace=ws_a)
        state["a"] = rd.rd_accept(lg, td["beams"], d["unpack_index"], d["n_packed"], out=state.get("a"), workspace=ws_c)

    def snapshot():
        torch.cuda.synchronize()
        s = {k: host(v) for k, v in state["d"].items()}
        s["o"] = host(state["o"])
        s.update({"acc_" + k: host(v) for k, v in state["a"].items()})
        return s

    step()
    eager = snapshot()
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            step()
    for rep in range(3):
        for v in list(state["d"].values()) + [state["o"]] + list(state["a"].values()):
            v.fill_(0) if v.dtype != torch.bfloat16 else v.zero_()      # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for k in eager:
            assert np.array_equal(got[k], eager[k]), (rep, k)


def _to_pages(t, ps, rng, extra=5):
    """Cuts the dense caches of case t into pages of ps keys scattered over a pool in random order."""
    kc, vc, ctx = t["k_cache"], t["v_cache"], t["ctx_len"]
    B, H, Cmax, D = kc.shape
    max_pages = max(1, -(-Cmax // ps))
    need = int(sum(-(-int(c) // ps) for c in ctx))
    n_pages = need + extra
    order = rng.permutation(n_pages)
    poison = synth.poison_value("bf16" if kc.dtype == np.uint16 else "f16")
    kp = np.full((n_pages, H, ps, D), poison, kc.dtype)
    vp = np.full((n_pages, H, ps, D), poison, kc.dtype)
    table = np.full((B, max_pages), -7, np.int32)
    nxt = 0
    for b in range(B):
        for j in range(-(-int(ctx[b]) // ps)):
            page = int(order[nxt]); nxt += 1
            table[b, j] = page
            n = min(ps, Cmax - j * ps)
            kp[page, :, :n] = kc[b, :, j * ps:j * ps + n]
            vp[page, :, :n] = vc[b, :, j * ps:j * ps + n]
    return kp, vp, table


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("ps", [32, 64, 128, 256])
@pytest.mark.parametrize("D,W,L,ctx", [(128, 8, 5, [0, 1, 31, 129, 300, 517]), (64, 16, 6, [700, 33]),
                                       (128, 70, 5, [97, 640]), (128, 16, 5, [5000, 2311])])
def test_paged_cache(rd, dtype, ps, D, W, L, ctx):
    """rd_tree_attn_paged against the oracle's paged routine: pages scattered over a pool, every
    page size, ragged contexts ending inside a page, wide beams, long contexts with several splits;
    unused rows of the pages and unused table entries hold poison."""
    announce("attn paged dtype=%s page=%d D=%d W=%d L=%d" % (dtype, ps, D, W, L))
    rng = np.random.default_rng(ps + D + W)
    t = make_case(len(ctx), 2, D, W, L, ctx, dtype, seed=ps + W, V=6)
    kp, vp, table = _to_pages(t, ps, rng)
    d = oracle.dedup(t["beams"], t["ctx_len"])
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn_paged(t["q"], kp, vp, np.maximum(table, 0), t["ctx_len"], t["k_new"], t["v_new"],
                                 d["n_packed"], d["tree_mask"], dtype, scale)
    got = rd.rd_tree_attn_paged(dev(t["q"]), dev(kp), dev(vp), dev(table), dev(t["ctx_len"]), dev(t["k_new"]),
                                dev(t["v_new"]), dev(d["n_packed"]), dev(d["tree_mask_bits"]), scale)
    torch.cuda.synchronize()
    compare(host(got), ref, dtype, "paged")


def test_paged_equals_dense_on_config2(rd):
    """Same bits as the dense entry point on the Vicuna-7B-shaped layer (the arithmetic is identical;
    only the addresses of the context tiles differ)."""
    announce("attn paged vs dense, config 2")
    cfg = synth.CONFIGS[2]
    t = synth.make_attn_inputs(cfg, poison=False)
    d = oracle.dedup(t["beams"], t["ctx_len"])
    scale = float(1.0 / np.sqrt(cfg.D))
    dense = gpu_attn(rd, t, d, cfg.dtype, scale)
    kp, vp, table = _to_pages(t, 128, np.random.default_rng(2))
    got = rd.rd_tree_attn_paged(dev(t["q"]), dev(kp), dev(vp), dev(table), dev(t["ctx_len"]), dev(t["k_new"]),
                                dev(t["v_new"]), dev(d["n_packed"]), dev(d["tree_mask_bits"]), scale)
    torch.cuda.synchronize()
    assert np.array_equal(host(got), dense)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_plan_from_a_context_bound(rd, dtype):
    """A cache allocated for 4096 keys holding contexts of a few hundred: rd_tree_attn_bounded plans for the
    bound the caller passes (exact, generous, or too small -- the bound steers the plan, never the result)
    and must give what rd_tree_attn gives; one workspace serves all the bounds."""
    announce("attn planned from a context bound, " + dtype)
    B, H, D, W, L, Cmax = 2, 8, 128, 8, 5, 4096
    ctx = np.array([600, 411], np.int32)
    t = make_case(B, H, D, W, L, ctx, dtype, seed=9, V=32000)
    for name in ("k_cache", "v_cache"):                      # the live rows at the front of a Cmax-row cache, poison behind
        full = np.full((B, H, Cmax, D), synth.poison_value(dtype), t[name].dtype)
        full[:, :, : t[name].shape[2]] = t[name]
        t[name] = full
    d = oracle.dedup(t["beams"], t["ctx_len"])
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                           d["n_packed"], d["tree_mask"], dtype, scale)
    td = {k: dev(v) for k, v in t.items()}
    npk, mask = dev(d["n_packed"]), dev(d["tree_mask_bits"])
    dt_code = rd.RD_BF16 if dtype == "bf16" else rd.RD_F32
    nbytes = max(rd.rd_tree_attn_workspace(B, H, W * L, D, c, dt_code) for c in (600, 1024, 300, 4096))
    ws = rd.new_workspace(nbytes, "cuda")
    base = rd.rd_tree_attn(td["q"], td["k_cache"], td["v_cache"], td["ctx_len"], td["k_new"], td["v_new"], npk, mask, scale)
    torch.cuda.synchronize()
    compare(host(base), ref, dtype, "capacity plan")
    for bound in (600, 1024, 300, 4096, 100000):
        got = rd.rd_tree_attn(td["q"], td["k_cache"], td["v_cache"], td["ctx_len"], td["k_new"], td["v_new"], npk, mask, scale,
                              workspace=ws, ctx_bound=bound)
        torch.cuda.synchronize()
        compare(host(got), ref, dtype, "bound %d" % bound)


@pytest.mark.parametrize("W", [30, 40])
def test_one_workspace_for_bounds_with_different_ranges(rd, W):
    """Beams of 150 or 200 tokens (four or five row groups) whose keys are split into more or fewer ranges, by the bound of the
    contexts: calls planned for alternating bounds share one workspace, as a decoding loop whose contexts grow does, and the
    arrival words of one plan must not lie where another has partial results."""
    announce("attn bounds with different ranges, W=%d" % W)
    B, H, D, L, Cmax, dtype = 2, 4, 128, 5, 4000, "bf16"
    N = W * L
    words = 8 * B * H * n_row_groups(N)
    bounds = (300, 4000, 300, 1000, 100, 4000, 1000, 300, 4000)
    need = {c: rd.rd_tree_attn_workspace(B, H, N, D, c, rd.RD_BF16) for c in bounds}
    assert len(set(need.values())) >= 3 and min(need.values()) > 2 * words      # several plans, all with partial results
    t = make_case(B, H, D, W, L, (Cmax, 410), dtype, seed=11, V=32000, share="high")
    d = oracle.dedup(t["beams"], t["ctx_len"])
    scale = float(1.0 / np.sqrt(D))
    ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"],
                           d["n_packed"], d["tree_mask"], dtype, scale)
    td = {k: dev(v) for k, v in t.items()}
    npk, mask = dev(d["n_packed"]), dev(d["tree_mask_bits"])
    ws = rd.new_workspace(max(need.values()), "cuda")
    for i, bound in enumerate(bounds):
        out = torch.full_like(td["q"], float("nan"))
        rd.rd_tree_attn(td["q"], td["k_cache"], td["v_cache"], td["ctx_len"], td["k_new"], td["v_new"], npk, mask, scale,
                        out=out, workspace=ws, ctx_bound=bound)
        torch.cuda.synchronize()
        compare(host(out), ref, dtype, "call %d, bound %d" % (i, bound))
        assert int(ws[:words].to(torch.int64).sum()) == 0


@pytest.mark.parametrize("bound", [300.0, "300", np.int64(300), np.float32(300.5), 2 ** 40, torch.tensor(300)])
def test_bound_and_scale_of_any_number_type(rd, bound):
    """ctx_bound is whatever int() takes and scale whatever float() takes; a bound beyond a C int is above every capacity."""
    announce("attn bound %r" % (bound,))
    B, H, D, W, L = 1, 2, 64, 3, 4
    t = make_case(B, H, D, W, L, [600], "bf16", seed=6)
    d = oracle.dedup(t["beams"], t["ctx_len"])
    ref = oracle.tree_attn(t["q"], t["k_cache"], t["v_cache"], t["ctx_len"], t["k_new"], t["v_new"], d["n_packed"], d["tree_mask"], "bf16", 0.125)
    args = [dev(t[k]) for k in ("q", "k_cache", "v_cache", "ctx_len", "k_new", "v_new")] + [dev(d["n_packed"]), dev(d["tree_mask_bits"])]
    for scale in (0.125, "0.125", np.float32(0.125)):
        got = rd.rd_tree_attn(*args, scale, ctx_bound=bound)
        torch.cuda.synchronize()
        compare(host(got), ref, "bf16", "bound %r, scale %r" % (bound, scale))
    with pytest.raises(rd.RdError):
        rd.rd_tree_attn(*args, 0.125, ctx_bound=-2 ** 40)
