"""Rotation and append of a prefill: in the epilogue of an unsplit QKV projection of tiles of 256 weight rows, by kernels behind it
otherwise.  The arithmetic is the same, so queries, keys and values are, bit for bit."""
import numpy as np
import pytest
import torch

from harness import workload as W
from stage_helpers import i32

pytestmark = pytest.mark.gpu


# Every tile that can rotate is an epilogue of its own.  (With 2560 + 1024 columns a last tile of the projection is half padding; odd
# lengths leave rows of the last tile over; with 29 heads and with 44 + 11 a wave's two heads of 64 channels are a query and a key, and a
# key and a value.)
@pytest.mark.parametrize("heads,kv_heads,dh,M,rows", [
    (16, 16, 128, 2567, 128), (16, 16, 128, 1407, 160), (16, 16, 128, 1703, 192), (16, 16, 128, 2001, 224), (16, 16, 128, 2505, 256),
    (20, 4, 128, 2431, 160), (32, 8, 64, 2815, 160), (32, 32, 64, 1500, 160),
    (44, 11, 64, 1823, 128), (29, 29, 64, 1501, 160), (44, 11, 64, 2503, 192), (29, 29, 64, 2203, 224), (44, 11, 64, 3407, 256),
])
@pytest.mark.parametrize("bias", [False, True])
def test_both_places_give_the_same_bits(heads, kv_heads, dh, M, rows, bias):
    """One layer in which every sum is exact: inputs of +-1 with rms_eps = 0, weights and biases in 16ths, the output projection the
    identity, no MLP.  The first prompts have to come out of a large call as they do out of a small one."""
    from paper_2506_10470_amd import tdp
    d, dkv, ff = heads * dh, kv_heads * dh, 128
    lens = np.array([1, 16, 33, 15, 100])
    first = int(lens.sum())
    n_qkv = -(-(d + 2 * dkv) // 256) * 256
    ways = [tdp.tdp_gemm_plan(m, n_qkv, d, 0, True, min(8 * 512 * max(n_qkv, d), 64 << 20)) for m in (first, M)]
    assert [p["splits"] == 1 and p["weight_rows"] == 256 for p in ways] == [False, True], ways
    assert ways[1]["rows"] == rows, ways
    rest = M - first
    all_lens = np.concatenate([lens, np.full(rest // 333, 333), [rest % 333]])
    g = torch.Generator(device="cuda").manual_seed(M)
    ints = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda").float() / 16
    w = {"wq": ints(d, d), "wk": ints(d, dkv), "wv": ints(d, dkv), "wo": torch.eye(d, device="cuda")}
    x = (torch.randint(0, 2, (M, d), generator=g, device="cuda") * 2 - 1).to(torch.bfloat16)
    tables, pages = W.block_tables(5, all_lens, max_pages_per_seq=22)
    st = tdp.tdp_stage_create(tdp.StageConfig(
        n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_ff=ff, rms_eps=0.0, rope_base=1e4,
        page_size=16, num_pages=pages, max_batch=0, max_tokens=M, max_seqs=len(all_lens), max_pages_per_seq=22))
    results = []
    try:
        for name, t in w.items():
            tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], t.to(torch.bfloat16), tdp.BF16, tdp.DEVICE, *t.shape)
        for name in ("g_attn", "g_mlp"):
            tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], torch.ones(d, device="cuda"), tdp.F32, tdp.DEVICE, d, 1)
        if bias:
            for name, n in (("bq", d), ("bk", dkv), ("bv", dkv)):
                b = torch.arange(n, device="cuda").remainder(7).float() / 16
                tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], b, tdp.F32, tdp.DEVICE, n, 1)
        for n in (len(lens), len(all_lens)):
            cu = np.concatenate([[0], np.cumsum(all_lens[:n])])
            T = int(cu[-1])
            out = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
            tdp.tdp_stage_prefill(st, x, i32(cu), i32(tables), n, T, out)
            k, v = (torch.empty((T, kv_heads, dh), dtype=torch.bfloat16, device="cuda") for _ in "kv")
            tdp.tdp_stage_kv_export(st, 0, k, v, i32(cu), i32(np.maximum(tables, 0)), n, T)
            torch.cuda.synchronize()
            assert not torch.isnan(out.float()).any()
            results.append([t[:first].clone().view(torch.int16) for t in (out, k, v)])
    finally:
        tdp.tdp_stage_destroy(st)
    for a, b in zip(*results):
        assert torch.equal(a, b)
