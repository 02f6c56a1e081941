"""Replay backward with chosen numbers of routes per expert: the token-contracted
weight gradients advance 32 routes a step through four LDS stages and hold 8192
route offsets at a time, the row-tile products 256 rows a tile.  The weights are the
paper-literal ones, whose dense router gradient is summed over chunks of 64 tokens
(96 at the largest case).

Every expert's slice of each expert-weight gradient is held to the bar of
tests/test_gpu_backward.py (Frobenius ratio <= 2e-2) by itself."""
import numpy as np
import pytest

import workloads as W
from tests import test_gpu_backward as TB

pytestmark = pytest.mark.gpu

STEPS = [0, 1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 160, 161, 255, 256, 257, 300]


@pytest.mark.parametrize("counts,d,m", [(STEPS, 256, 256), (STEPS, 512, 384),
                                        ([8193, 5, 8192, 0], 256, 128)],
                         ids=["steps", "steps_half_panel", "offset_chunks"])
def test_route_counts(counts, d, m):
    T, N = sum(counts), len(counts)
    s = W.LayerShape("counts", T=T, d=d, N=N, k=1, m=m, r=0, act="bf16", skew="none")
    L = W.layer_inputs(s, 23)
    idx = np.random.default_rng(23).permutation(np.repeat(np.arange(N), counts)).reshape(T, 1)
    dy = W.upstream_grad(s, 23)
    g = TB.run_bwd(L, idx, dy, "bf16", renorm=False)
    ref = TB.oracle_bwd(L, idx, dy, renorm=False)
    TB.compare(g, ref, "bf16", f"{N} experts, d {d}, m {m}")
    for n in ("dW_gate", "dW_up", "dW_down"):
        for e, c in enumerate(counts):
            if c == 0:
                assert np.all(g[n][e] == 0.0)
            else:
                err = TB.frob(g[n][e], ref[n][e])
                assert err <= TB.TOL["bf16"], f"{n} of expert {e} ({c} routes): {err:.2e}"
