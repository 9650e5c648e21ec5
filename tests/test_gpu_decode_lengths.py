"""Decode steps at lengths where the sharing-out of a context changes: requests of many spans, and ctx_lens that do not fit their
block-table rows.  The kernels bring such a length into the row's range, so every access stays inside the tables, the work list
and the grid, and the counters of finished spans end where they began: what the step leaves behind is one overwritten slot
of the request's own pages, and later steps are not affected."""
import numpy as np
import pytest
import torch

from harness import workload as W
from harness.runner import Stage, i32
from test_gpu_parity import run_decode_case

pytestmark = pytest.mark.gpu

WIDTH, SPAN = 40, 256           # 640 tokens per row: three spans at most


@pytest.mark.parametrize("shape", ["tiny_gqa", "tiny_h128"])
@pytest.mark.parametrize("span", [SPAN, 1024])  # with a work list, and (one span per request) without one
def test_lengths_outside_a_row_leave_later_steps_alone(shape, span):
    from paper_2506_10470_amd import tdp
    sh = W.SHAPES[shape].with_layers(2)
    good = np.array([0, 300, 639, 17, 511])
    bad = np.array([2 ** 31 - 1, 640, 100000, -5, -2 ** 31])
    B = len(good)
    tables = np.random.default_rng(3).permutation(B * WIDTH).reshape(B, WIDTH)
    x = W.hidden_states(sh, B, 1, device="cuda")
    full = i32(np.arange(B + 1) * WIDTH * 16)
    total = B * WIDTH * 16

    def fill(st):
        for l in range(sh.n_layers):
            k, v = (W.kv_packed(sh, l, w, total, 7, device="cuda") for w in "kv")
            tdp.tdp_stage_kv_import(st.h, l, k, v, full, i32(tables), B, total)

    def step(st, ctx):
        out = torch.full_like(x, float("nan"))
        tdp.tdp_stage_decode(st.h, x, i32(ctx.astype(np.int64).astype(np.int32)), i32(tables), B, out)
        torch.cuda.synchronize()
        return out.view(torch.int16)

    with Stage(tdp, sh, B * WIDTH, B, 0, 0, WIDTH) as st:
        tdp.tdp_stage_set_decode_span(st.h, span)
        fill(st)
        expected = step(st, good)
    with Stage(tdp, sh, B * WIDTH, B, 0, 0, WIDTH) as st:
        tdp.tdp_stage_set_decode_span(st.h, span)
        fill(st)
        before = [tuple(t.clone() for t in st.pools(l)) for l in range(sh.n_layers)]
        step(st, bad)
        for l in range(sh.n_layers):
            k, v = st.pools(l)
            changed_k = (k.view(torch.int16) != before[l][0].view(torch.int16)).any(dim=3).any(dim=1)  # [page][slot]
            changed_v = (v.view(torch.int16) != before[l][1].view(torch.int16)).any(dim=2).any(dim=1)
            allowed = torch.zeros_like(changed_k)
            for b in range(B):
                pos = min(max(int(bad[b]), 0), WIDTH * 16 - 1)
                allowed[tables[b, pos // 16], pos % 16] = True
            assert not (changed_k & ~allowed).any() and not (changed_v & ~allowed).any()
        fill(st)
        for _ in range(2):
            assert torch.equal(step(st, good), expected)


@pytest.mark.parametrize("q_heads,kv_heads,head_dim", [(2, 2, 64), (2, 2, 128), (6, 2, 128), (10, 2, 64), (16, 2, 128)])
def test_many_spans_are_combined_by_all_threads(q_heads, kv_heads, head_dim):
    """More than 16 spans are shared out in runs where a group of heads leaves threads over: 16, 8, 2, 3 and (none left) 1 run,
    with 16 spans (still one), 17 and 40, and a request of one span beside them."""
    from paper_2506_10470_amd import tdp
    sh = W.StageShape("spans", 1, 256, q_heads, kv_heads, head_dim, 128)
    run_decode_case(tdp, sh, [4095, 4096, 10000, 3], max_pages_per_seq=626, span=256)


@pytest.mark.parametrize("group,head_dim,kv_scales", [(1, 64, None), (1, 128, (0.03125, 0.7)), (2, 128, None), (2, 64, (0.03125, 0.7))])
def test_both_ways_of_combining_spans_give_the_same_bits(group, head_dim, kv_scales):
    """With one or two query heads per K/V head, how long a context the block tables allow decides whether spans are combined by
    the attention kernel (9216 tokens: nine spans of 1024) or by a kernel behind it (10240: ten).  The order of the spans is the
    same, so the outputs are."""
    from paper_2506_10470_amd import tdp
    heads, ctx = 40, np.array([5000, 0, 1023, 1024, 9215, 3, 2047, 2048, 100, 1500, 4096])
    sh = W.StageShape("ways", 1, 256, group * heads, heads, head_dim, 128)
    B = len(ctx)
    x = W.hidden_states(sh, B, 1, device="cuda")
    cu = np.concatenate([[0], np.cumsum(ctx)])
    outs = []
    for tokens in (9216, 10240):
        tables, pages = W.block_tables(9, ctx + 1, max_pages_per_seq=tokens // 16)
        with Stage(tdp, sh, pages, B, 0, 0, tokens // 16, kv_scales=kv_scales) as st:
            for l in range(sh.n_layers):
                k, v = (W.kv_packed(sh, l, w, int(cu[-1]), 7, device="cuda") for w in "kv")
                tdp.tdp_stage_kv_import(st.h, l, k, v, i32(cu), i32(np.maximum(tables, 0)), B, int(cu[-1]))
            out = torch.full_like(x, float("nan"))
            tdp.tdp_stage_timing_enable(st.h, True)
            tdp.tdp_stage_decode(st.h, x, i32(ctx), i32(tables), B, out)
            assert (tdp.tdp_stage_timing_read(st.h)["attention_merge"] > 0) == (tokens == 10240)
            outs.append(out.view(torch.int16))
    assert not torch.isnan(out.float()).any()
    assert torch.equal(*outs)
