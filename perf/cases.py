"""The work that a decoding program has this library do, as cases that can be timed and compared.

Three kinds of call sequence, all through `paper_2403_09919_amd.binding`:

  step    the verification of one decoding step for `layers` decoder layers: rd_dedup once, attention once per
          layer (each layer with its own cache, as in a model), rd_accept once and, with `commit`, the accepted
          rows appended to every layer's cache and the hidden state of the last accepted token picked out.
  draft   rd_draft: the draft model and its beam search.
  sample  rd_accept_sample: acceptance by rejection sampling.

Shapes come from the five synthetic configurations (`synth.CONFIGS`), from the drafter sizes that go with them and
from the widest beams of the paper's sweep; `draw` spreads over the same ranges.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2403_09919_amd import binding as rd
from paper_2403_09919_amd import synth

_ESZ = {"f32": 4, "bf16": 2, "f16": 2}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _step(name, B, ctx_lo, ctx_hi, H, D, dtype, W, L, V, share="uniform", layers=1, rope=False, commit=False, cache="dense",
          page=0, bound=False, capacity=0, root=False, lean=True, launch="eager"):
    """`capacity`: positions allocated per sequence (0: what the longest context and one step need); `bound`: the
    caller hands over the longest live context; `lean`: no dense mask and no prefix tree asked of rd_dedup."""
    return dict(name=name, kind="step", B=B, ctx_lo=ctx_lo, ctx_hi=ctx_hi, H=H, D=D, dtype=dtype, W=W, L=L, V=V, share=share,
                layers=layers, rope=rope, commit=commit, cache=cache, page=page, bound=bound, capacity=capacity,
                root=root, lean=lean, launch=launch)


def _draft(name, B, W, L, Dm, V, n_mlp=2, dtype="bf16", tiled=True, steps=False):
    return dict(name=name, kind="draft", B=B, W=W, L=L, Dm=Dm, V=V, n_mlp=n_mlp, dtype=dtype, tiled=tiled, steps=steps)


def _sample(name, B, W, L, V, record, root=False, temperature=0.8):
    return dict(name=name, kind="sample", B=B, W=W, L=L, V=V, record=record, root=root, temperature=temperature)


def listed():
    return [
        # a toy model in fp32: every call is a few microseconds, so latency and host time are all there is
        _step("tiny_f32", 1, 128, 128, 4, 64, "f32", 4, 4, 1000, lean=False),
        # one interactive user on a 7B-shaped model: a whole decoding step over its 32 layers, launched from Python
        _step("interactive_7b_model", 1, 1024, 1024, 32, 128, "bf16", 8, 5, 32000, layers=32, rope=True, commit=True),
        # one layer of the same model replayed from a HIP graph: the benchmark's headline step
        _step("interactive_7b_graph", 1, 1024, 1024, 32, 128, "bf16", 8, 5, 32000, lean=False, launch="graph"),
        # a batch of ragged contexts on the 7B shape
        _step("batched_7b_ragged", 8, 1024, 2048, 32, 128, "bf16", 8, 5, 32000, layers=4, rope=True, commit=True),
        # few sequences with long contexts on the 13B shape, the first token verified as well
        _step("long_13b", 4, 4096, 4096, 40, 128, "bf16", 16, 5, 32000, layers=2, root=True, commit=True),
        # throughput serving on the 33B shape with beams that share most of their prefixes: the largest verification
        _step("batched_33b", 16, 2048, 2048, 52, 128, "bf16", 16, 5, 32000, share="high"),
        # continuous batching in fp16: many short ragged sequences in a paged cache, narrow beams
        _step("paged_serving_f16", 24, 101, 1500, 32, 128, "f16", 5, 5, 32000, layers=4, commit=True, cache="paged", page=64),
        # the widest beam of the paper's sweep (70 candidates of 5 tokens), cache capacity far above the live context
        _step("wide_beam_7b", 1, 1777, 1777, 32, 128, "bf16", 70, 5, 32000, layers=8, bound=True, capacity=4096),
        # the drafter of an interactive user, of a small batch that samples (it keeps the record of the search) and of a large one
        _draft("draft_7b_one_user", 1, 8, 5, 4096, 32000),
        _draft("draft_13b_batch", 4, 16, 5, 5120, 32000, steps=True),
        _draft("draft_33b_batch", 16, 16, 5, 6656, 32000, dtype="f16"),
        # sampling at a temperature, the draft distributions read from the drafter's own record
        _sample("sampling_7b_batch", 8, 8, 5, 32000, record=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("step", "step", "step", "draft", "sample"))
        W = _log_int(rng, 1, 70)
        L = rng.randint(2, 8)
        B = _log_int(rng, 1, 24)
        if W * L > 384:
            continue
        if kind == "draft":
            if B * W > 256:
                continue
            c = _draft("", B, W, L, 64 * _log_int(rng, 8, 104), _log_int(rng, 4000, 64000), rng.randint(1, 3),
                       rng.choice(("bf16", "f16")), rng.random() < 0.75, rng.random() < 0.3)
            top = _work_draft(listed()[10])["bytes"]
        elif kind == "sample":
            c = _sample("", B, W, L, _log_int(rng, 4000, 128000), rng.random() < 0.5, rng.random() < 0.3,
                        round(rng.uniform(0.5, 1.2), 3))
            top = 4e8
        else:
            hi = _log_int(rng, 64, 6000)
            lo = hi if rng.random() < 0.4 else max(1, int(hi * rng.uniform(0.1, 0.9)))
            dtype = rng.choice(("bf16", "bf16", "f16", "f32"))
            half = dtype != "f32"
            cache = "paged" if half and rng.random() < 0.25 else "dense"
            c = _step("", B, lo, hi, rng.choice((4, 5, 8, 10, 16, 26, 32, 40, 52)), rng.choice((64, 128, 128)), dtype, W, L,
                      _log_int(rng, 4000, 64000), rng.choice(("uniform", "high")), _log_int(rng, 1, 32),
                      half and cache == "dense" and rng.random() < 0.4, rng.random() < 0.5, cache,
                      rng.choice((32, 64, 128)) if cache == "paged" else 0, False, 0, rng.random() < 0.3, rng.random() < 0.7,
                      rng.choice(("eager", "eager", "graph")))
            if cache == "dense" and not c["rope"] and rng.random() < 0.3:
                c["bound"], c["capacity"] = True, hi + 8 + rng.randint(0, 3 * hi)
            top, most = (1e9, 6e10) if half else (4e7, 2e9)     # fp32 is the exactness path, not the serving one
            while c["layers"] > 1 and (_work_step(c)["bytes"] > top or _work_step(c)["flops"] > most):
                c["layers"] //= 2
            if _work_step(c)["flops"] > most:
                continue
        if work(c)["bytes"] <= top:
            del c["name"]
            return c


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _plant(logits, d, seed, p_plant, bump):
    """The LLM usually agrees with one of the drafted continuations: with probability p_plant a child of a packed node
    gets `bump` on its token."""
    rng = np.random.default_rng(int(seed))
    parent, tokens, n_packed = (d[k].cpu().numpy() for k in ("parent", "packed_tokens", "n_packed"))
    rows, toks = [], []
    for b in range(parent.shape[0]):
        kids = {}
        for c in range(int(n_packed[b])):
            kids.setdefault(int(parent[b, c]), []).append(c)
        for p, cs in kids.items():
            u, k = rng.random(), int(rng.integers(0, len(cs)))
            if p >= 0 and u < p_plant:
                rows.append((b, p))
                toks.append(int(tokens[b, cs[k]]))
    if rows:
        r = torch.tensor(rows, device="cuda")
        logits[r[:, 0], r[:, 1], torch.tensor(toks, device="cuda")] += bump


def _roots(beams, seed):
    """The LLM's own first token: the best candidate's in three sequences of four."""
    rng = np.random.default_rng([int(seed), 77])
    root = beams[:, 0, 0].copy()
    root[rng.random(root.shape[0]) < 0.25] += 1
    return torch.from_numpy(root).cuda()


def _prepare_step(c, seed):
    B, H, D, W, L, V, layers = (c[k] for k in ("B", "H", "D", "W", "L", "V", "layers"))
    N, dt, gen = W * L, _TORCH[c["dtype"]], _generator(seed)

    def randn(*shape, dtype=dt):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)

    beams_np = synth.make_beams(B, W, L, V, seed, c["share"])
    ctx_np = synth.make_ctx_len(B, c["ctx_lo"], c["ctx_hi"], seed)
    s = dict(c, beams=torch.from_numpy(beams_np).cuda(), ctx_len=torch.from_numpy(ctx_np).cuda(), scale=1.0 / math.sqrt(D))
    s["root_token"] = _roots(beams_np, seed) if c["root"] else None
    s["ctx_bound"] = int(ctx_np.max()) if c["bound"] else None
    for name in ("q", "k_new", "v_new"):
        s[name] = randn(layers, B, H, N, D)
    cap = max(c["capacity"], c["ctx_hi"] + L)
    code = {"f32": rd.RD_F32, "bf16": rd.RD_BF16, "f16": rd.RD_F16}[c["dtype"]]
    if c["cache"] == "paged":
        per = -(-cap // c["page"])
        s["block_table"] = torch.randperm(B * per, generator=gen, device="cuda").to(torch.int32).view(B, per)
        shape = (layers, B * per, H, c["page"], D)
        need = rd.rd_tree_attn_paged_workspace(B, H, N, D, c["page"], per, code)
    else:
        shape = (layers, B, H, cap, D)
        need = rd.rd_tree_attn_workspace(B, H, N, D, min(cap, s["ctx_bound"] or cap), code)
    s["k_cache"], s["v_cache"] = randn(*shape), randn(*shape)
    s["attn_ws"], s["accept_ws"] = rd.new_workspace(need, "cuda"), rd.new_workspace(rd.rd_accept_workspace(B, W, L, V), "cuda")
    s["attn_out"] = torch.empty_like(s["q"])
    if c["rope"]:
        ang = torch.outer(torch.arange(cap + L, device="cuda", dtype=torch.float32),
                          10000.0 ** (-torch.arange(0, D, 2, device="cuda", dtype=torch.float32) / D))
        s["cos"], s["sin"] = ang.cos(), ang.sin()
        s["k_rot"] = torch.zeros_like(s["k_new"])
    if c["commit"]:
        s["ctx_next"], s["n_committed"] = torch.zeros_like(s["ctx_len"]), torch.zeros_like(s["ctx_len"])
        s["hidden"] = randn(B, N, H * D) if c["cache"] == "dense" else None
        s["hidden_last"] = torch.zeros((B, H * D), dtype=dt, device="cuda") if c["cache"] == "dense" else None
    s["dedup"] = rd.rd_dedup(s["beams"], s["ctx_len"], want_prefix_tree=not c["lean"], want_mask=not c["lean"])
    s["logits"] = randn(B, N, V, dtype=torch.float32)
    _plant(s["logits"], s["dedup"], seed, 0.7, 8.0)
    s["accept"] = dict(argmax=torch.empty((B, N), dtype=torch.int32, device="cuda"),
                       n_accept=torch.empty((B, W), dtype=torch.int32, device="cuda"),
                       accepted_idx=torch.empty((B, L), dtype=torch.int32, device="cuda"),
                       **{k: torch.empty((B,), dtype=torch.int32, device="cuda") for k in ("best_beam", "best_len", "next_token")})
    # a program holds one tensor per layer, not one that it slices on each step
    for name in ("q", "k_new", "v_new", "k_cache", "v_cache", "attn_out") + (("k_rot",) if c["rope"] else ()):
        s[name + "_of"] = list(s[name].unbind(0))
    if c["launch"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _run_step(s)
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _run_step(s)
    return s


def _prepare_draft(c, seed):
    B, W, L, Dm, V, K, dt, gen = c["B"], c["W"], c["L"], c["Dm"], c["V"], c["n_mlp"], _TORCH[c["dtype"]], _generator(seed)
    G = 2 * Dm

    def randn(shape, std=1.0, dtype=dt):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype).mul_(std)

    # What a trained drafter has and random matrices lack: LLM hidden states share a direction from which the output
    # layer reads each token's frequency, and the state carries what went before along another (`turn`; with f = SiLU
    # and entries of +-1 the component along it is halved, hence 1 and 2 below).  Without such directions candidates
    # lie closer together than 16-bit activations can tell apart.
    common, turn = randn((Dm,), 1.0, torch.float32), torch.sign(randn((Dm,), 1.0, torch.float32))
    emb, head = randn((V, Dm), 0.8), randn((V, G), 0.1 * G ** -0.5)
    kind, follows = randn((V,), 0.6, torch.float32), randn((V,), 2.0, torch.float32)
    rank = torch.randperm(V, generator=gen, device="cuda").float()
    for at in range(0, V, 8192):
        of = slice(at, at + 8192)
        emb[of] = emb[of].float() + torch.outer(kind[of], turn)
        head[of, :Dm] = head[of, :Dm].float() + torch.outer(follows[of], turn / Dm)
        head[of, Dm:] = head[of, Dm:].float() + torch.outer(20.0 - 4.0 * torch.log1p(rank[of]), common / Dm)
    rnn_u, rnn_w = (randn((Dm, Dm), Dm ** -0.5) + (g * torch.outer(turn, turn / Dm)).to(dt) for g in (1.0, 2.0))
    params = dict(emb=emb, rnn_u=rnn_u, rnn_w=rnn_w, rnn_b=randn((Dm,), 0.01, torch.float32),
                  mlp_w=randn((K, G, G), G ** -0.5), mlp_b=randn((K, G), 0.01, torch.float32), head_w=head)
    if c["tiled"]:
        params = rd.rd_draft_pack(params)
    out = dict(beams=torch.empty((B, W, L), dtype=torch.int32, device="cuda"),
               beam_logp=torch.empty((B, W), dtype=torch.float32, device="cuda"))
    if c["steps"]:
        out["step_logits"] = torch.zeros((L - 1, B * W, V), dtype=torch.float32, device="cuda")
        out["step_row"] = torch.zeros((B, W, L - 1), dtype=torch.int32, device="cuda")
    return dict(c, params=params, h=(0.8 * common + randn((B, Dm), 0.6, torch.float32)).to(dt),
                last_token=torch.randint(0, V, (B,), generator=gen, device="cuda", dtype=torch.int32), out=out,
                ws=torch.empty(rd.rd_draft_workspace(B, W, L, Dm, V), dtype=torch.uint8, device="cuda"))


def _prepare_sample(c, seed):
    B, W, L, V, gen = c["B"], c["W"], c["L"], c["V"], _generator(seed)
    N = W * L
    beams_np = synth.make_beams(B, W, L, V, seed)
    s = dict(c, beams=torch.from_numpy(beams_np).cuda(), root_token=_roots(beams_np, seed) if c["root"] else None)
    d = s["dedup"] = rd.rd_dedup(s["beams"])
    # peaked as an LLM's: a few tokens hold most of the probability
    logits = torch.randn((B, N, V), generator=gen, device="cuda").mul_(4.0)
    _plant(logits, d, seed, 0.7, 18.0)
    s["logits"], s["step_row"] = logits, None
    if c["record"]:          # one row per live candidate and position, shared by the candidates with that prefix
        s["step_row"] = (d["prefix_tree"][:, :, :L - 1] + W * torch.arange(B, device="cuda", dtype=torch.int32).view(B, 1, 1)).contiguous()
        draft = torch.empty((L - 1, B * W, V), device="cuda")
        for j in range(L - 1):
            at = d["unpack_index"][:, :, j].long()
            draft[j] = logits[torch.arange(B, device="cuda").view(B, 1), at].view(B * W, V)
    else:
        draft = logits.clone()
    s["draft_logits"] = draft.add_(torch.randn(draft.shape, generator=gen, device="cuda"))
    s["u_accept"] = torch.rand((B, N), generator=gen, device="cuda")
    s["u_next"] = torch.rand((B,), generator=gen, device="cuda")
    s["out"] = dict(n_accept=torch.empty((B, W), dtype=torch.int32, device="cuda"),
                    accepted_idx=torch.empty((B, L), dtype=torch.int32, device="cuda"),
                    **{k: torch.empty((B,), dtype=torch.int32, device="cuda") for k in ("best_beam", "best_len", "next_token")})
    s["ws"] = rd.new_workspace(rd.rd_accept_sample_workspace(B, W, L, V), "cuda")
    return s


def prepare(case, seed):
    return {"step": _prepare_step, "draft": _prepare_draft, "sample": _prepare_sample}[case["kind"]](case, seed)


# ------------------------------------------------------------------------------------------
# the calls
# ------------------------------------------------------------------------------------------
def _run_step(s):
    d = rd.rd_dedup(s["beams"], s["ctx_len"], out=s["dedup"])
    n_packed, bits, scale, ws = d["n_packed"], d["tree_mask_bits"], s["scale"], s["attn_ws"]
    paged, rope = s["cache"] == "paged", s["rope"]
    for i in range(s["layers"]):
        q, k, v = s["q_of"][i], s["k_new_of"][i], s["v_new_of"][i]
        kc, vc, out = s["k_cache_of"][i], s["v_cache_of"][i], s["attn_out_of"][i]
        if paged:
            rd.rd_tree_attn_paged(q, kc, vc, s["block_table"], s["ctx_len"], k, v, n_packed, bits, scale, out=out, workspace=ws)
        elif rope:
            rd.rd_tree_attn_rope(q, kc, vc, s["ctx_len"], k, v, n_packed, bits, d["position_ids"], s["cos"], s["sin"], scale,
                                 out=out, k_new_rot=s["k_rot_of"][i], workspace=ws)
        else:
            rd.rd_tree_attn(q, kc, vc, s["ctx_len"], k, v, n_packed, bits, scale, out=out, workspace=ws, ctx_bound=s["ctx_bound"])
    acc = rd.rd_accept(s["logits"], s["beams"], d["unpack_index"], n_packed, s["root_token"], out=s["accept"], workspace=s["accept_ws"])
    if s["commit"]:
        idx, best = acc["accepted_idx"], acc["best_len"]
        last = s["layers"] - 1
        for i in range(s["layers"]):
            k = s["k_rot_of"][i] if rope else s["k_new_of"][i]
            if paged:
                rd.rd_commit_paged(k, s["v_new_of"][i], idx, best, s["ctx_len"], s["k_cache_of"][i], s["v_cache_of"][i],
                                   s["block_table"], ctx_len_out=s["ctx_next"], n_committed=s["n_committed"])
            elif i < last:
                rd.rd_commit(k, s["v_new_of"][i], idx, best, s["ctx_len"], s["k_cache_of"][i], s["v_cache_of"][i],
                             ctx_len_out=s["ctx_next"], n_committed=s["n_committed"])
            else:
                rd.rd_commit(k, s["v_new_of"][i], idx, best, s["ctx_len"], s["k_cache_of"][i], s["v_cache_of"][i],
                             ctx_len_out=s["ctx_next"], n_committed=s["n_committed"], hidden=s["hidden"],
                             hidden_last=s["hidden_last"])


def run(s):
    if s["kind"] == "draft":
        return rd.rd_draft(s["params"], s["h"], s["last_token"], s["W"], s["L"], out=s["out"], workspace=s["ws"])
    if s["kind"] == "sample":
        return rd.rd_accept_sample(s["logits"], s["draft_logits"], s["beams"], s["dedup"]["unpack_index"], s["dedup"]["n_packed"],
                                   s["u_accept"], s["u_next"], s["temperature"], root_token=s["root_token"], out=s["out"],
                                   workspace=s["ws"], step_row=s["step_row"])
    if "graph" in s:
        s["graph"].replay()
    else:
        _run_step(s)
    got = dict(s["dedup"], attn_out=s["attn_out"], **s["accept"])
    if s["rope"]:
        got["k_rot"] = s["k_rot"]
    if s["commit"]:
        got.update(k_cache=s["k_cache"], v_cache=s["v_cache"], ctx_next=s["ctx_next"], n_committed=s["n_committed"],
                   hidden_last=s["hidden_last"])
    return got


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _packed(B, W, L, V, share):
    """Distinct prefixes in the batch: (all of them, those that are not whole candidates), for one draw of the beams."""
    beams = synth.make_beams(B, W, L, V, 1, share)
    inner = sum(len({tuple(cand[:j]) for cand in seq}) for seq in beams.tolist() for j in range(1, L))
    return inner + sum(len({tuple(cand) for cand in seq}) for seq in beams.tolist()), inner


def _work_step(c):
    B, H, D, e = c["B"], c["H"], c["D"], _ESZ[c["dtype"]]
    P, _ = _packed(B, c["W"], c["L"], c["V"], c["share"])
    keys = B * (c["ctx_lo"] + c["ctx_hi"]) / 2
    # per layer: each live cache entry read once, packed q, k, v read and the output written once
    per_layer = e * H * D * (2 * keys + 4 * P)
    flops = 4.0 * H * D * P * (keys / B + 2.5)
    return {"bytes": c["layers"] * per_layer + 4.0 * P * c["V"], "flops": c["layers"] * flops}


def _work_draft(c):
    # every drafted position depends on the one before and the weights exceed every cache: they are read once per
    # position (the RNN's from the second on)
    Dm, V, K, n = c["Dm"], c["V"], c["n_mlp"], c["L"] - 1
    dense, rnn = K * 4 * Dm * Dm + 2 * Dm * V, 2 * Dm * Dm
    rows = c["B"] + (n - 1) * c["B"] * c["W"]
    record = 4.0 * rows * V if c["steps"] else 0.0
    return {"bytes": 2.0 * (n * dense + (n - 1) * rnn) + record,
            "flops": 2.0 * (rows * dense + (rows - c["B"]) * rnn)}


def work(case):
    if case["kind"] == "draft":
        return _work_draft(case)
    if case["kind"] == "sample":
        P, inner = _packed(case["B"], case["W"], case["L"], case["V"], "uniform")
        return {"bytes": 4.0 * case["V"] * (P + inner), "flops": 0.0}
    return _work_step(case)


def tolerance(case):
    if case["kind"] == "sample":          # a draw within rounding of its threshold may go the other way
        return {"rel": 0.0, "differ": 0.01}
    if case["kind"] == "draft":
        # fp32 sums in another order move single 16-bit activations by one unit in the last place, and candidates
        # that lie closer than that may swap
        return {"rel": 1e-2, "differ": 0.01}
    # attention: storage type of the probabilities and of the result; everything else is copied or whole numbers
    return {"f32": {"rel": 1e-5, "max": 1e-4}, "f16": {"rel": 2e-3, "max": 0.02}, "bf16": {"rel": 1e-2, "max": 0.1}}[case["dtype"]]
