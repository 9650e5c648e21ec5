"""Rotation and append of a decode step: inside the attention kernel while all (request, K/V head) pairs run at once and spans of 256
tokens are not too many, by a kernel in front of it beyond that.  The arithmetic is the same, so what is stored and attended to is, bit for bit."""
import numpy as np
import pytest
import torch

from harness import workload as W
from stage_helpers import i32

pytestmark = pytest.mark.gpu
PAIRS = 768          # the most that are rotated inside


@pytest.mark.parametrize("heads,kv_heads,dh,scales", [
    (8, 8, 64, None), (8, 8, 128, (0.03125, 0.7)), (4, 2, 128, None), (10, 2, 64, None), (16, 2, 128, None),
    (16, 1, 64, None), (16, 1, 128, None), (13, 1, 64, (0.5, 0.02)), (16, 2, 128, (0.03125, 0.7)),
])
@pytest.mark.parametrize("bias", [False, True])
def test_both_places_give_the_same_bits(heads, kv_heads, dh, scales, bias):
    """One layer in which every sum is exact, so that a request's result cannot depend on the batch around it: inputs of +-1 with
    rms_eps = 0, weights and biases in 16ths, the output projection the identity, no MLP.  The first requests of a batch of
    exactly PAIRS pairs, of a small one and of one that is larger have to come out alike: first slots of pages and last ones,
    an empty context, more than one span."""
    from paper_2506_10470_amd import tdp
    d, dkv, ff, width = heads * dh, kv_heads * dh, 128, 80
    ctx = np.array([0, 15, 16, 31, 33, 127, 1200, 300, 255, 256])
    sizes = [len(ctx), PAIRS // kv_heads, PAIRS // kv_heads + 1]
    g = torch.Generator(device="cuda").manual_seed(heads * dh + kv_heads)
    ints = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda").float() / 16
    w = {"wq": ints(d, d), "wk": ints(d, dkv), "wv": ints(d, dkv), "wo": torch.eye(d, device="cuda")}
    most = sizes[-1]
    x = (torch.randint(0, 2, (most, d), generator=g, device="cuda") * 2 - 1).to(torch.bfloat16)
    all_ctx = np.concatenate([ctx, np.arange(most - len(ctx)) % 40])
    tables, pages = W.block_tables(5, all_ctx + 1, max_pages_per_seq=width)
    cu = np.concatenate([[0], np.cumsum(all_ctx)])
    total = int(cu[-1])
    k, v = (torch.randn(total, kv_heads, dh, generator=g, device="cuda").to(torch.bfloat16) for _ in "kv")
    results = []
    for B in sizes:
        st = tdp.tdp_stage_create(tdp.StageConfig(
            n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_ff=ff, rms_eps=0.0, rope_base=1e4,
            page_size=16, num_pages=pages, max_batch=most, max_tokens=0, max_seqs=0, max_pages_per_seq=width,
            kv_dtype=tdp.KV_FP8_E4M3 if scales else tdp.KV_BF16, k_scale=scales[0] if scales else 0.0,
            v_scale=scales[1] if scales else 0.0))
        try:
            for name, t in w.items():
                tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], t.to(torch.bfloat16), tdp.BF16, tdp.DEVICE, *t.shape)
            for name in ("g_attn", "g_mlp"):
                tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], torch.ones(d, device="cuda"), tdp.F32, tdp.DEVICE, d, 1)
            if bias:
                for name, n in (("bq", d), ("bk", dkv), ("bv", dkv)):
                    b = torch.arange(n, device="cuda").remainder(7).float() / 16
                    tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], b, tdp.F32, tdp.DEVICE, n, 1)
            tdp.tdp_stage_set_decode_span(st, 1024)
            tdp.tdp_stage_kv_import(st, 0, k, v, i32(cu), i32(np.maximum(tables, 0)), most, total)
            out = torch.full((B, d), float("nan"), dtype=torch.bfloat16, device="cuda")
            tdp.tdp_stage_timing_enable(st, True)
            tdp.tdp_stage_decode(st, x, i32(all_ctx), i32(tables), B, out)
            torch.cuda.synchronize()
            assert (tdp.tdp_stage_timing_read(st)["rope_kv"] > 0) == (B * kv_heads > PAIRS)
            full = i32(np.concatenate([[0], np.cumsum(all_ctx + 1)]))
            n = total + most
            ko, vo = (torch.empty((n, kv_heads, dh), dtype=torch.bfloat16, device="cuda") for _ in "kv")
            tdp.tdp_stage_kv_export(st, 0, ko, vo, full, i32(np.maximum(tables, 0)), most, n)
            torch.cuda.synchronize()
            first = int((ctx + 1).sum())
            results.append([t.clone().view(torch.int16) for t in (out[:len(ctx)], ko[:first], vo[:first])])
        finally:
            tdp.tdp_stage_destroy(st)
    assert not torch.isnan(out.float()).any()
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("spans,inside", [(128, True), (129, False)])   # of 256 tokens that a block-table row has room for
@pytest.mark.parametrize("scales", [None, (0.03125, 0.7)])
def test_many_short_spans_are_rotated_in_front(spans, inside, scales):
    """64 pairs of requests whose block tables allow 8192 or 8256 workgroups; the same requests give the same bits either way."""
    from paper_2506_10470_amd import tdp
    B, heads, kv_heads, dh = 32, 4, 2, 64
    d, dkv = heads * dh, kv_heads * dh
    ctx = np.array([0, 255, 256, 700, 1500] + [11] * (B - 5))
    cu, total = i32(np.concatenate([[0], np.cumsum(ctx)])), int(ctx.sum())
    g = torch.Generator(device="cuda").manual_seed(3)
    w = {n: (torch.randn(*s, generator=g, device="cuda") * 0.1).to(torch.bfloat16)
         for n, s in (("wq", (d, d)), ("wk", (d, dkv)), ("wv", (d, dkv)), ("wo", (d, d)))}
    x = torch.randn(B, d, generator=g, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn(total, kv_heads, dh, generator=g, device="cuda").to(torch.bfloat16) for _ in "kv")
    outs = []
    for width in (128, spans * 16):
        tables, pages = W.block_tables(5, ctx + 1, max_pages_per_seq=width)
        st = tdp.tdp_stage_create(tdp.StageConfig(
            n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_ff=128, rms_eps=1e-5, rope_base=1e4,
            page_size=16, num_pages=pages, max_batch=B, max_tokens=0, max_seqs=0, max_pages_per_seq=width,
            kv_dtype=tdp.KV_FP8_E4M3 if scales else tdp.KV_BF16, k_scale=scales[0] if scales else 0.0,
            v_scale=scales[1] if scales else 0.0))
        try:
            for name, t in w.items():
                tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], t, tdp.BF16, tdp.DEVICE, *t.shape)
            for name in ("g_attn", "g_mlp"):
                tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], torch.ones(d, device="cuda"), tdp.F32, tdp.DEVICE, d, 1)
            tdp.tdp_stage_kv_import(st, 0, k, v, cu, i32(np.maximum(tables, 0)), B, total)
            out = torch.full((B, d), float("nan"), dtype=torch.bfloat16, device="cuda")
            tdp.tdp_stage_timing_enable(st, True)
            tdp.tdp_stage_decode(st, x, i32(ctx), i32(tables), B, out)
            torch.cuda.synchronize()
            assert (tdp.tdp_stage_timing_read(st)["rope_kv"] == 0) == (inside or width == 128)
            outs.append(out.view(torch.int16))
        finally:
            tdp.tdp_stage_destroy(st)
    assert not torch.isnan(out.float()).any() and torch.equal(*outs)
