"""Prefill attention at the edges of its blocks: 64 tokens of a block, 32 of a half, 16 of a page, 8 of a lane's load, in pools whose
other slots hold NaN."""
import numpy as np
import pytest
import torch

from harness import workload as W
from oracle import stage_oracle as O
from stage_helpers import Stage, f64, i32, oracle_layers
from test_gpu_fp8_kv import q8_shape, row_errs, row_tolerances
from test_gpu_parity import run_prefill_case, tdp  # noqa: F401

pytestmark = pytest.mark.gpu


LENGTHS = [1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 95, 97, 127, 128, 129, 191, 193, 257]


@pytest.mark.parametrize("heads,kv_heads,dh", [(2, 2, 64), (2, 2, 128), (10, 2, 64), (16, 2, 128)])
def test_prompts_that_end_beside_an_edge(tdp, heads, kv_heads, dh):
    sh = W.StageShape("edges", 1, 256, heads, kv_heads, dh, 128)
    run_prefill_case(tdp, sh, LENGTHS)


@pytest.mark.parametrize("heads,kv_heads,dh", [(2, 2, 64), (2, 2, 128), (10, 2, 64), (16, 2, 128)])
def test_the_same_with_an_8_bit_cache(tdp, heads, kv_heads, dh):
    """Values past a prompt's end are cleared behind the conversion; a NaN that is left reaches every row of its block."""
    sh, scales = W.StageShape("edges", 1, 256, heads, kv_heads, dh, 128), (1.0, 0.5)
    lens = np.array(LENGTHS)
    n, T = len(lens), int(lens.sum())
    cu = np.concatenate([[0], np.cumsum(lens)])
    pb = W.make_prefill_batch(lens)
    with Stage(tdp, sh, pb.num_pages, n, T, n, pb.tables.shape[1], kv_scales=scales) as st:
        st.poison()
        x = W.hidden_states(sh, T, 2, device="cuda")
        out = torch.empty_like(x)
        tdp.tdp_stage_prefill(st.h, x, i32(cu), i32(pb.tables), n, T, out)
        torch.cuda.synchronize()
        xs = f64(x)
        ref, _ = O.stage_prefill([xs[a:b] for a, b in zip(cu, cu[1:])], list(oracle_layers(sh)), q8_shape(sh, scales))
        errs = row_errs(f64(out), np.concatenate(ref))
        assert np.all(errs <= row_tolerances(np.concatenate([np.arange(L) for L in lens]))), float(np.max(errs))
