"""The few-rows expert GEMMs (decode batches) against the 256-row tiles: a small
batch's outputs must be bitwise those of the same tokens in a batch that is over the
kernels' routes-per-expert limits, at the edges of their 8-row copies, 16-row MFMA
tiles and 64-row workgroups.  Parity with the oracle is tests/test_gpu_replay.py's."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_replay import dev_layer, run_replay

pytestmark = pytest.mark.gpu

CASES = [
    # (N, k, d, m, small T, routes of expert 0)
    (64, 1, 256, 128, 150, (1, 7, 8, 9, 15, 16, 17)),
    (128, 1, 512, 192, 400, (31, 32, 33, 48, 49, 63, 64, 65)),
    (256, 2, 256, 384, 300, (128, 129, 255, 256, 257)),
    # fewer work items than XCDs, and ranges that the XCDs do not share evenly
    (4, 1, 256, 128, 40, (1, 2, 39, 40)),
    (13, 1, 768, 640, 100, (1, 65, 100)),
]


@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}_k{c[1]}_d{c[2]}_m{c[3]}" for c in CASES])
def test_few_rows_match_tiles(case):
    N, k, d, m, T, heads = case
    big = 40 * N // k + T
    s = W.LayerShape("few", T=big, d=d, N=N, k=k, m=m, r=0, act="bf16", skew="none")
    L = W.layer_inputs(s, 41)
    D = dev_layer(L, "bf16")
    rng = np.random.default_rng(41)
    for n0 in heads:
        # the first n0 tokens route to expert 0, the others away from it
        idx = 1 + np.argsort(rng.random((big, N - 1)), axis=1)[:, :k].astype(np.int32)
        idx[:n0, 0] = 0
        y, g = run_replay(D, idx)
        ys, gs = run_replay(D, idx[:T], x=D["x"][:T])
        np.testing.assert_array_equal(gs, g[:T], err_msg=f"weights, {n0} routes of expert 0")
        np.testing.assert_array_equal(ys, y[:T], err_msg=f"outputs, {n0} routes of expert 0")
