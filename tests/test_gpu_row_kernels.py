"""Small kernels around the projections at the sizes where they change shape: the greedy selection on rows of any
alignment and length, the decode plan and the rotation + append for batches above the 256 threads of a plan."""
import numpy as np
import pytest
import torch

from test_gpu_parity import run_decode_case, tdp  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 511, 515, 1023, 2048, 2051, 4099, 5003, 16383, 19999, 20003, 32768, 32771, 70001])
def test_argmax_any_alignment(tdp, n):
    """Rows ld apart start at every offset inside 16 bytes; few distinct values, so ties are everywhere."""
    M, ld = 9, n + 5 if n % 2 else n + 3
    rng = np.random.default_rng(n)
    x = rng.integers(-2, 3, size=(M, ld)).astype(np.float32)
    x[1, :n] = -np.inf
    x[2, :n] = np.nan
    x[3, :n], x[3, n - 1] = np.nan, -np.inf
    x[4, n - 1] = 7.0
    x[:, n:] = 100.0
    out = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    tdp.tdp_argmax_rows(torch.from_numpy(x).cuda(), M, n, ld, out)
    v = np.where(np.isnan(x[:, :n]), -np.inf, x[:, :n])
    ref = v.argmax(axis=1)
    ref[3] = n - 1  # the only number of its row
    assert np.array_equal(out.cpu().numpy(), ref)


@pytest.mark.parametrize("shape,n", [("tiny_gqa", 257), ("tiny_h128", 600)])
def test_decode_of_more_requests_than_a_plan_has_threads(tdp, shape, n):
    rng = np.random.default_rng(n)
    ctx = rng.integers(0, 40, size=n)
    ctx[::97] = rng.integers(200, 900, size=len(ctx[::97]))   # several spans of the shortest span length
    run_decode_case(tdp, shape, ctx)
