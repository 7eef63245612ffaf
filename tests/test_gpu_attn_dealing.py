"""The ways in which the 16-bit attention kernel deals a batch's heads to its workgroups, against the oracle: ragged contexts in no
order, with equal lengths and a 0 among them, and packed counts that differ from sequence to sequence, in dense and paged
caches and with the rotation inside the call."""
import numpy as np
import pytest
import torch

import oracle
from attn_dealing import SHAPES
from gpu_util import announce, dev, host
from paper_2403_09919_amd import synth
from test_gpu_attn import _to_pages
from test_gpu_attn_edges import TOL
from test_oracle_rope import tables

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rd():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2403_09919_amd import binding
    return binding


@pytest.mark.parametrize("kind", ["dense", "paged", "rope"])
@pytest.mark.parametrize("way,B,H,W,L,D,C", SHAPES)
def test_dealing(rd, kind, way, B, H, W, L, D, C):
    announce(f"dealing {way} {kind} B={B} H={H} W={W} L={L} D={D} C={C}")
    dtype = "f16" if kind == "paged" else "bf16"
    rng = np.random.default_rng(B + H)
    ctx = rng.integers(1, C + 1, B).astype(np.int32)
    ctx[rng.integers(0, B, 3)] = [C, 0, C]                          # (at least one of the longest)
    ctx[-1] = C
    ctx[1] = ctx[B // 2]
    # few and many distinct prefixes: 1, 2 or 32000 tokens to choose from
    beams = np.concatenate([synth.make_beams(1, W, L, int(rng.choice([1, 2, 32000])), i, "uniform") for i in range(B)])
    N, scale = W * L, float(1.0 / np.sqrt(D))
    q, kn, vn = synth.make_qkv_new(B, H, N, D, dtype, B)
    kc, vc = synth.make_kv_cache(B, H, C, D, dtype, B, ctx, True)
    d = oracle.dedup(beams, ctx)
    npk, bits = dev(d["n_packed"]), dev(d["tree_mask_bits"])
    out = torch.full_like(dev(q), float("nan"))
    if kind == "rope":
        cos, sin = tables(C + L, D)
        q2, k2 = dev(q), dev(kn)
        rd.rd_rope(q2, k2, dev(d["position_ids"]), npk, dev(cos), dev(sin))
        ref = oracle.tree_attn(host(q2), kc, vc, ctx, host(k2), vn, d["n_packed"], d["tree_mask"], dtype, scale)
        _, k_rot = rd.rd_tree_attn_rope(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), npk, bits, dev(d["position_ids"]), dev(cos), dev(sin),
                                        scale, out=out)
        torch.cuda.synchronize()
        for b in range(B):
            P = int(d["n_packed"][b])
            assert np.array_equal(host(k_rot[b, :, :P]), host(k2[b, :, :P]))
    else:
        ref = oracle.tree_attn(q, kc, vc, ctx, kn, vn, d["n_packed"], d["tree_mask"], dtype, scale)
        if kind == "paged":
            # 32 keys a page, and as many pages per sequence as the dense cache has keys for: the same launch plan
            kp, vp, table = _to_pages(dict(k_cache=kc, v_cache=vc, ctx_len=ctx), 32, rng)
            rd.rd_tree_attn_paged(dev(q), dev(kp), dev(vp), dev(table), dev(ctx), dev(kn), dev(vn), npk, bits, scale, out=out)
        else:
            rd.rd_tree_attn(dev(q), dev(kc), dev(vc), dev(ctx), dev(kn), dev(vn), npk, bits, scale, out=out)
        torch.cuda.synchronize()
    got, want = synth.to_f64(host(out), dtype), synth.to_f64(ref, dtype)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL[dtype]
    for b in range(B):
        assert not got[b, :, int(d["n_packed"][b]):].any()
