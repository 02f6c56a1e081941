"""Replay backward of bf16 layers whose expert width is a multiple of 128 but not
of 256: the down projection's gradient products then end in a half panel.

Oracle, bar (Frobenius ratio <= 2e-2 per tensor) and recorded routes are those of
tests/test_gpu_backward.py; the saved-pre-activation pass must be bitwise the
recomputing one."""
import numpy as np
import pytest

import workloads as W
from tests import test_gpu_backward as TB
from tests import test_gpu_saved as TS

pytestmark = pytest.mark.gpu

CASES = [
    # (T, d, N, k, m, skew, idx_dtype, ldi_pad, renorm)
    (301, 256, 8, 2, 128, "hot8", "int32", 0, True),      # a single half panel
    (700, 512, 16, 4, 384, "zipf", "int16", 3, True),
    (257, 256, 64, 8, 640, "none", "int32", 0, False),    # experts with few or no rows
    (150, 2048, 8, 6, 1408, "none", "int32", 0, True),
    # one route past a tile of 64 rows.  (Not fewer tokens: a token's dp = g1 g2 (dg1 - dg2)
    # has the relative error 4e-3 (|dg1| + |dg2|) / |dg1 - dg2|, bounded in the mean over
    # tokens only; a single token showed 3.1e-2.)
    (65, 256, 4, 2, 384, "none", "int32", 0, True),
]


@pytest.mark.parametrize("case", CASES, ids=[f"T{c[0]}_d{c[1]}_N{c[2]}_k{c[3]}_m{c[4]}"
                                              for c in CASES])
def test_half_panel(case):
    T, d, N, k, m, skew, idt, pad, renorm = case
    s = W.LayerShape("half", T=T, d=d, N=N, k=k, m=m, r=0, act="bf16", skew=skew, flip_frac=0.05)
    L = W.layer_inputs(s, 19)
    idx = TB.recorded_route(L, s, 19)
    dy = W.upstream_grad(s, 19)
    g = TB.run_bwd(L, idx, dy, "bf16", idt, pad, renorm=renorm)
    TB.compare(g, TB.oracle_bwd(L, idx, dy, renorm), "bf16", str(case))
    unused = np.setdiff1d(np.arange(N), np.unique(idx))
    for n in ("dW_gate", "dW_up", "dW_down"):
        assert np.all(g[n][unused] == 0.0), f"{n} of unused experts {unused} is not zero"
    TS.run_pair(L, s, idx, dy, renorm, idt, pad)
