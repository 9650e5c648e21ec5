"""KV import / export page by page against the element-by-element path (taken for packed arrays that are not 16-byte
aligned): the pools and the packed arrays have to be the same, bit for bit, poison outside the written slots included."""
import numpy as np
import pytest
import torch

from harness import workload as W
from stage_helpers import Stage, i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdp():
    from paper_2506_10470_amd import tdp as _tdp
    return _tdp


LENS = [1, 15, 16, 17, 48, 0, 33, 7]
MANY = LENS + [4096, 1, 4097, 2900]      # 690 pages: more workgroups of 512 channels than run at once ("wide")


@pytest.mark.parametrize("kv_scales", [None, (0.03125, 0.7)])
@pytest.mark.parametrize("shape,seq_lens", [("tiny_gqa", LENS), ("tiny", LENS), ("tiny_g2", LENS), ("wide", LENS), ("wide", MANY),
                                            ("tiny_gqa", MANY)])
def test_page_moves_equal_the_element_path(tdp, shape, seq_lens, kv_scales):
    sh = W.SHAPES["tiny"] if shape == "wide" else W.SHAPES[shape]
    if shape == "wide":   # 1280 channels: three column blocks, the last one half full
        sh = W.StageShape("wide", 1, 256, 10, 10, 128, 64)
    lens = np.array(seq_lens, dtype=np.int64)
    tab, pages = W.block_tables(77, lens)
    cu = np.concatenate([[0], np.cumsum(lens)])
    total, ch = int(cu[-1]), sh.n_kv_heads * sh.head_dim
    g = torch.Generator(device="cpu").manual_seed(5)
    k = torch.randn(total * ch, generator=g).to(torch.bfloat16)
    v = torch.randn(total * ch, generator=g).to(torch.bfloat16)
    k[3], v[5] = float("nan"), float("inf")

    def on_gpu(x, shift):
        b = torch.zeros(total * ch + 8, dtype=torch.bfloat16, device="cuda")
        b[shift:shift + total * ch] = x.cuda()
        return b, b[shift:shift + total * ch]

    got = []
    with Stage(tdp, sh, pages, 1, 0, 0, tab.shape[1], load_weights=False, kv_scales=kv_scales) as st:
        for shift in (0, 1):
            st.poison()
            (kb, kd), (vb, vd) = on_gpu(k, shift), on_gpu(v, shift)
            tdp.tdp_stage_kv_import(st.h, 0, kd, vd, i32(cu), i32(tab), len(lens), total)
            torch.cuda.synchronize()
            pools = [p.clone() for p in st.raw_pools(0)]
            (ob, ok), (pb, ov) = on_gpu(torch.zeros_like(k), shift), on_gpu(torch.zeros_like(v), shift)
            tdp.tdp_stage_kv_export(st.h, 0, ok, ov, i32(cu), i32(tab), len(lens), total)
            torch.cuda.synchronize()
            got.append([t.contiguous().view(torch.uint8).cpu() for t in (pools[0], pools[1], ok.clone(), ov.clone())])
            assert ob[total * ch + shift:].abs().sum() == 0 and pb[total * ch + shift:].abs().sum() == 0
    for a, b in zip(*got):
        assert torch.equal(a, b)
    if kv_scales is None:
        assert torch.equal(got[0][2], k.view(torch.uint8)) and torch.equal(got[0][3], v.view(torch.uint8))


def test_a_prefix_of_the_packed_tokens_can_be_moved(tdp):
    """total_tokens below the last prefix sum: only those tokens move, as token by token."""
    sh = W.SHAPES["tiny_gqa"]
    lens = np.array([20, 30], dtype=np.int64)
    tab, pages = W.block_tables(78, lens)
    cu = i32(np.concatenate([[0], np.cumsum(lens)]))
    k = torch.randn(50, sh.n_kv_heads, sh.head_dim, device="cuda").to(torch.bfloat16)
    with Stage(tdp, sh, pages, 1, 0, 0, tab.shape[1], load_weights=False) as st:
        for total in (13, 20, 37):
            out = torch.zeros_like(k)
            st.poison()
            tdp.tdp_stage_kv_import(st.h, 0, k, k, cu, i32(tab), 2, total)
            tdp.tdp_stage_kv_export(st.h, 0, out, torch.zeros_like(k), cu, i32(tab), 2, total)
            torch.cuda.synchronize()
            assert torch.equal(out[:total], k[:total]) and out[total:].abs().sum() == 0
            kf, _ = st.raw_pools(0)
            assert int((~torch.isnan(kf.float())).sum()) == total * sh.n_kv_heads * sh.head_dim


@pytest.mark.parametrize("kv_scales", [None, (0.03125, 0.7)])
@pytest.mark.parametrize("tokens", [3276, 3277, 13107, 13108, 52428, 52429])   # 1280 channels: one token below and from 16, 64, 256 MiB on
def test_large_moves_equal_the_element_path(tdp, tokens, kv_scales):
    lens = [4095] * (tokens // 4095) + [tokens % 4095]
    test_page_moves_equal_the_element_path(tdp, "wide", lens, kv_scales)
