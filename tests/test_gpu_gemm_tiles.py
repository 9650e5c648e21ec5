"""The projection GEMM against the fp64 product and, bit for bit, one way of making it against another: every tile that
there is, forced, over several lengths of its ring of k-stages; the tiles that the plan takes; split-K and chunked sums, also
where the last part is a short one; and the sums that a stage leaves to the rotation and to the norm.  Operands are exact in bf16
and sums are fp32, so what separates a result from the fp64 product is the rounding of the output, 2^-9 of its magnitude,
and the fp32 sum, far below: 1e-2 of the row maximum as everywhere in these tests."""
import functools

import numpy as np
import pytest
import torch

from harness.runner import dev_view_bf16, i32
from stage_helpers import f64, row_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdp():
    from paper_2506_10470_amd import tdp as _tdp
    return _tdp


# number of a tile: (rows, weight rows, slots of its ring, sums in chunks)
TILES = {1: (256, 256, 4, False), 2: (128, 256, 6, False), 3: (128, 128, 4, False), 4: (224, 256, 4, False), 5: (192, 256, 5, False),
         6: (160, 256, 5, False), 7: (256, 128, 6, False), 8: (224, 128, 6, False), 9: (160, 128, 7, False), 10: (96, 128, 8, True),
         11: (128, 128, 9, True), 12: (64, 128, 6, True), 13: (32, 128, 4, True)}
N_FORCED, K_FORCED = 1032, 23 * 64   # ragged columns; 46 stages: five to eleven rings, and a multiple of no ring


@functools.lru_cache(maxsize=None)
def problem(M, N, K, epi):
    """A, W, R on the GPU, and the fp64 result."""
    g = torch.Generator(device="cpu").manual_seed(M * 31 + N)
    A = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    Wm = (torch.randn(K, N, generator=g) * (2.0 / K ** 0.5)).to(torch.bfloat16).cuda()
    cols = N // 2 if epi == 2 else N
    R = torch.randn(M, cols, generator=g).to(torch.bfloat16).cuda()
    ref = (A.double() @ Wm.double()).cpu().numpy()
    if epi == 1:
        ref = ref + f64(R)
    if epi == 2:
        gate = ref[:, :cols]
        ref = gate / (1.0 + np.exp(-gate)) * ref[:, cols:]
    return A, Wm, (R if epi == 1 else None), cols, ref


def made(tdp, M, N, K, epi, tile, splits=1, chunk_k=0):
    A, Wm, R, cols, _ = problem(M, N, K, epi)
    out = torch.full((M, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    tdp.tdp_gemm_bf16_form(A, Wm, R, out, M, N, K, epi, tile, splits, chunk_k)
    return out


@pytest.mark.parametrize("tile", TILES)
def test_forced_tile_over_several_rings(tdp, tile):
    """All tiles add a (split's) K range up in the same order, so they agree with 256 x 256 to the bit; that one is held to the
    fp64 product.  A stage read too early, or a slot filled over one that is still read, shows in either."""
    rows, _, slots, _ = TILES[tile]
    stages = K_FORCED // 32
    assert stages % slots and stages > 5 * slots
    for M in (1, rows - 1, rows + 1, 2 * rows + 33):
        for epi in (0, 1, 2):
            for splits in (1, 3):   # 23 k-tiles: 8 + 8 + 7
                got, base = (made(tdp, M, N_FORCED, K_FORCED, epi, t, splits) for t in (tile, 1))
                assert torch.equal(got.view(torch.int16), base.view(torch.int16)), (M, epi, splits)
                assert row_rel_err(f64(got), problem(M, N_FORCED, K_FORCED, epi)[4]) <= 1e-2, (M, epi, splits)


@pytest.mark.parametrize("tile", [t for t in TILES if TILES[t][3]])
@pytest.mark.parametrize("chunk,splits", [(8, 3), (5, 5), (12, 2), (22, 2), (1, 23), (23, 1)])
def test_chunked_sums_equal_the_split_ones(tdp, tile, chunk, splits):
    """k-tiles per chunk, and how many chunks that makes of 23: the last one is shorter, up to one k-tile of 23."""
    assert -(-23 // chunk) == splits
    rows = TILES[tile][0]
    for M in (1, rows, rows + 5):
        for epi in (0, 2):
            got = made(tdp, M, N_FORCED, K_FORCED, epi, tile, 1, chunk * 64)
            if chunk == 22:  # (a split factor deals K out evenly, 12 + 11: compared with the fp64 product alone)
                assert row_rel_err(f64(got), problem(M, N_FORCED, K_FORCED, epi)[4]) <= 1e-2
            else:
                assert torch.equal(got.view(torch.int16), made(tdp, M, N_FORCED, K_FORCED, epi, 2, splits).view(torch.int16))


def test_forms_that_do_not_exist_are_refused(tdp):
    A, Wm, _, _, _ = problem(1, N_FORCED, K_FORCED, 0)
    out = torch.empty((1, N_FORCED), dtype=torch.bfloat16, device="cuda")
    for tile, splits, chunk_k in [(0, 1, 0), (14, 1, 0), (1, 0, 0), (1, 24, 0), (1, 9, 0), (1, 1, 64), (12, 2, 64), (12, 1, 32)]:
        with pytest.raises(tdp.TdpError) as e:
            tdp.tdp_gemm_bf16_form(A, Wm, None, out, 1, N_FORCED, K_FORCED, 0, tile, splits, chunk_k)
        assert e.value.code == tdp.EINVAL


SHAPES = [
    # M, N, K, and the tile that the plan takes
    (450, 30008, 128, (256, 256)),
    (385, 30008, 128, (224, 256)),   # two rows of tiles
    (700, 30008, 128, (192, 256)),   # four
    (257, 30008, 128, (160, 256)),   # two
    (255, 30008, 128, (256, 128)),
    (193, 30008, 128, (224, 128)),
    (129, 30008, 128, (160, 128)),
    (225, 8200, 2048, (96, 128)),    # three
    (128, 30008, 128, (128, 128)),
    (129, 8200, 2048, (64, 128)),
    (1, 8200, 2048, (32, 128)), (31, 520, 1024, (32, 128)), (33, 1032, 512, (32, 128)),
    (1301, 520, 192, (32, 128)),     # many short rows of tiles: bands of unequal height
]


@pytest.mark.parametrize("M,N,K,tile", SHAPES)
@pytest.mark.parametrize("epi,splits", [(0, 0), (1, 0), (2, 0), (0, 2), (2, 2)])
def test_planned_tiles_match_the_fp64_product(tdp, M, N, K, tile, epi, splits):
    """(With a split factor given, the plan may take another tile.)"""
    if splits == 0:
        p = tdp.tdp_gemm_plan(M, N, K, epi)
        assert (p["rows"], p["weight_rows"]) == tile
    g = torch.Generator(device="cpu").manual_seed(M * 31 + N)
    A = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    Wm = (torch.randn(K, N, generator=g) * (2.0 / K ** 0.5)).to(torch.bfloat16).cuda()
    cols = N // 2 if epi == 2 else N
    R = torch.randn(M, cols, generator=g).to(torch.bfloat16).cuda()
    out = torch.full((M, cols), float("nan"), dtype=torch.bfloat16, device="cuda")
    tdp.tdp_gemm_bf16(A, Wm, R if epi == 1 else None, out, M, N, K, epi, 0, splits)
    ref = (A.double() @ Wm.double()).cpu().numpy()
    if epi == 1:
        ref = ref + f64(R)
    if epi == 2:
        gate = ref[:, :cols]
        ref = gate / (1.0 + np.exp(-gate)) * ref[:, cols:]
    assert row_rel_err(f64(out), ref) <= 1e-2


@pytest.mark.parametrize("M,N,K,epi,splits,chunked", [
    # summed in chunks by one workgroup: equal ones, then a short last one
    (48, 22016, 4096, 2, 2, True), (1, 22016, 4096, 2, 2, True), (100, 27648, 5120, 2, 2, True), (128, 15360, 5120, 0, 4, True),
    (96, 22016, 4096, 2, 2, True), (48, 24576, 8192, 2, 5, True), (1, 12288, 2048, 2, 5, True),
    # split-K workgroups
    (33, 4096, 4096, 1, 16, False), (16, 8192, 2048, 1, 8, False), (64, 10240, 4096, 0, 6, False), (96, 4096, 14336, 1, 16, False),
])
def test_small_batches_keep_the_order_of_their_sums(tdp, M, N, K, epi, splits, chunked):
    """Up to 128 rows the plan may choose the tile but not the order of the sums: the result is bit for bit that of 128 x 256
    tiles with the split-K factor of the rule.  It differs from that of one factor less, or the test would show nothing (one
    more may be the same schedule: 64 k-tiles in 17 parts of 4 are 16 parts)."""
    p = tdp.tdp_gemm_plan(M, N, K, epi)
    assert (p["splits"], p["chunk_k"]) == ((1, -(-K // 64 // splits) * 64) if chunked else (splits, 0))
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    Wm = (torch.randn(K, N, generator=g, device="cuda") * (2.0 / K ** 0.5)).to(torch.bfloat16)
    cols = N // 2 if epi == 2 else N
    R = torch.randn(M, cols, generator=g, device="cuda").to(torch.bfloat16)

    def run(tile, s):
        out = torch.empty((M, cols), dtype=torch.bfloat16, device="cuda")
        tdp.tdp_gemm_bf16(A, Wm, R if epi == 1 else None, out, M, N, K, epi, tile, s)
        return out.view(torch.int16)

    planned = run(0, 0)
    assert torch.equal(planned, run(2, splits))
    assert not torch.equal(planned, run(2, splits - 1))


@pytest.mark.parametrize("M,heads,kv_heads", [(128, 40, 40), (48, 32, 32), (100, 40, 8), (17, 64, 8), (33, 16, 16), (200, 40, 40)])
def test_sums_left_to_the_rotation_and_the_norm(tdp, M, heads, kv_heads):
    """A stage's split QKV projection is summed by the rotation, its split O projection by the norm behind it, both in split
    order.  Seen through one layer in which nothing else rounds: inputs of +-1 with rms_eps = 0 leave the first norm as they are,
    position 0 is not turned and attends to its own value alone, and the MLP is zero.  So the pools hold K and V, and the
    output x + V * Wo, to the bit as one GEMM with the same split factor makes them."""
    dh, ff = 128, 128
    d, dkv = heads * dh, kv_heads * dh
    n_qkv = d + 2 * dkv
    workspace = min(8 * ((M + 1) & ~1) * max(-(-n_qkv // 256) * 256, d, 2 * ff), 64 << 20)
    g = torch.Generator(device="cuda").manual_seed(M + d)
    w = {n: (torch.randn(d, c, generator=g, device="cuda") * (2.0 / d ** 0.5)).to(torch.bfloat16)
         for n, c in (("q", d), ("k", dkv), ("v", dkv), ("o", d))}
    x = (torch.randint(0, 2, (M, d), generator=g, device="cuda") * 2 - 1).to(torch.bfloat16)
    ones = torch.ones(d, device="cuda")
    st = tdp.tdp_stage_create(tdp.StageConfig(
        n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_ff=ff, rms_eps=0.0, rope_base=1e4,
        page_size=16, num_pages=M, max_batch=M, max_tokens=0, max_seqs=0, max_pages_per_seq=1))
    try:
        for name in "qkvo":
            tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS["w" + name], w[name], tdp.BF16, tdp.DEVICE, *w[name].shape)
        for name in ("g_attn", "g_mlp"):
            tdp.tdp_stage_set_weight(st, 0, tdp.WEIGHT_IDS[name], ones, tdp.F32, tdp.DEVICE, d, 1)
        out = torch.empty_like(x)
        tdp.tdp_stage_decode(st, x, i32(np.zeros(M)), i32(np.arange(M)[:, None]), M, out)
        torch.cuda.synchronize()
        kp, vp, nbytes = tdp.tdp_stage_kv_pool(st, 0)
        # slot 0 of every request's page, from the documented layout
        k = dev_view_bf16(kp, nbytes).view(M, kv_heads, dh // 32, 16, 32)[:, :, :, 0].reshape(M, dkv).clone()
        v = dev_view_bf16(vp, nbytes).view(M, kv_heads, dh, 16)[..., 0].reshape(M, dkv).clone()
    finally:
        tdp.tdp_stage_destroy(st)

    def gemm(a, b, residual, n, plan):
        assert plan["splits"] > 1
        r = torch.empty((M, n), dtype=torch.bfloat16, device="cuda")
        tdp.tdp_gemm_bf16_form(a, b, residual, r, M, n, b.shape[0], 0 if residual is None else 1, 2, plan["splits"])
        return r

    qkv = gemm(x, torch.cat([w["q"], w["k"], w["v"]], dim=1).contiguous(), None, n_qkv,
               tdp.tdp_gemm_plan(M, n_qkv, d, 0, True, workspace))
    assert torch.equal(k.view(torch.int16), qkv[:, d:d + dkv].contiguous().view(torch.int16))
    assert torch.equal(v.view(torch.int16), qkv[:, d + dkv:].contiguous().view(torch.int16))
    attended = v.view(M, kv_heads, 1, dh).expand(M, kv_heads, heads // kv_heads, dh).reshape(M, d).contiguous()
    ref = gemm(attended, w["o"], x, d, tdp.tdp_gemm_plan(M, d, d, 1, True, workspace))
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
