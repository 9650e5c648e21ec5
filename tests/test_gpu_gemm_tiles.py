"""Every tile of the projection GEMM that the planner can choose, against the fp64 product: rows in steps of 32 (M
one past and one short of a step, several rows of tiles, unequal bands), 128 and 256 weight rows, ragged N, all
epilogues, with and without split-K.  Operands are exact in bf16 and sums are fp32, so what separates the result from
the fp64 product is the rounding of the output, 2^-9 of its magnitude, and the fp32 sum, far below: 1e-2 of the row maximum
as everywhere in these tests."""
import numpy as np
import pytest
import torch

from stage_helpers import f64, row_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tdp():
    from paper_2506_10470_amd import tdp as _tdp
    return _tdp


SHAPES = [
    # (M, N, K): the tile that the plan takes
    (450, 30008, 128),   # 256 x 256
    (385, 30008, 128),   # 224 x 256, two rows of tiles
    (700, 30008, 128),   # 192 x 256, four rows
    (257, 30008, 128),   # 160 x 256, two rows
    (255, 30008, 128),   # 256 x 128
    (193, 30008, 128),   # 224 x 128
    (129, 30008, 128),   # 160 x 128
    (225, 8200, 2048),   # 96 x 128, three rows
    (128, 30008, 128),   # 128 x 128, two workgroups per CU
    (129, 8200, 2048),   # 64 x 128
    (1, 8200, 2048), (31, 520, 1024), (33, 1032, 512),   # 32 x 128
    (1301, 520, 192),    # many short rows of tiles: bands of unequal height
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("epi,splits", [(0, 0), (1, 0), (2, 0), (0, 2), (2, 2)])
def test_every_tile_matches_the_fp64_product(tdp, M, N, K, epi, splits):
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


@pytest.mark.parametrize("M,N,K,epi,splits", [
    (48, 22016, 4096, 2, 2), (1, 22016, 4096, 2, 2), (100, 27648, 5120, 2, 2),   # summed in chunks by one workgroup
    (128, 15360, 5120, 0, 4), (33, 4096, 4096, 1, 16), (16, 8192, 2048, 1, 8),   # split-K workgroups
])
def test_small_batches_keep_the_order_of_their_sums(tdp, M, N, K, epi, splits):
    """Up to 128 rows the plan may choose the tile but not the order of the sums: the result is bit for bit that of 128 x 256
    tiles with the split-K factor of the rule.  It differs from that of one factor less, or the test would show nothing (one
    more may be the same schedule: 64 k-tiles in 17 parts of 4 are 16 parts)."""
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
