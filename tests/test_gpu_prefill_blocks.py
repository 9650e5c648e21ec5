"""Prefill attention at the edges of its blocks: 64 tokens of a block, 32 of a half, 16 of a page, 8 of a lane's load, in pools whose
other slots hold NaN."""
import pytest

from harness import workload as W
from test_gpu_parity import run_prefill_case, tdp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads,dh", [(2, 2, 64), (2, 2, 128), (10, 2, 64), (16, 2, 128)])
def test_prompts_that_end_beside_an_edge(tdp, heads, kv_heads, dh):
    sh = W.StageShape("edges", 1, 256, heads, kv_heads, dh, 128)
    run_prefill_case(tdp, sh, [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 95, 97, 127, 128, 129, 191, 193, 257])
