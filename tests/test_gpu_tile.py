"""The fp32-FMA tile kernels (fp32 layers, and bf16 layers that no MFMA kernel
takes) and the few-column form of the fp64 router, at the edges of their 64 x 64
tiles, 32-wide K steps and 64 columns, against the oracle.

Bars: gates and fp32 outputs <= 1e-5 relative (tests/test_gpu_replay.py), fp32
gradients <= 1e-4, bf16 <= 2e-2 (tests/test_gpu_backward.py)."""
import numpy as np
import pytest

from oracle import pr2_oracle as O
import workloads as W
from tests import test_gpu_backward as TB
from tests import test_gpu_replay as TR
from tests import test_gpu_saved as TS
from tests.parity import compare_gates, compare_rows

pytestmark = pytest.mark.gpu

CASES = [
    # (T, d, N, k, m, act): odd sizes (no wide loads), tile and step edges, 64 and 65 columns
    (65, 33, 3, 2, 65, "f32"),
    (129, 64, 5, 1, 64, "f32"),
    (300, 68, 2, 2, 132, "f32"),
    (31, 1, 64, 3, 1, "f32"),
    (40, 31, 65, 4, 32, "f32"),
    (200, 320, 8, 2, 96, "bf16"),
    (90, 63, 4, 3, 30, "bf16"),
]


@pytest.mark.parametrize("renorm", [True, False], ids=["renorm", "literal"])
@pytest.mark.parametrize("case", CASES, ids=[f"T{c[0]}_d{c[1]}_N{c[2]}_k{c[3]}_m{c[4]}_{c[5]}"
                                              for c in CASES])
def test_tile_kernels(case, renorm):
    T, d, N, k, m, act = case
    s = W.LayerShape("tile", T=T, d=d, N=N, k=k, m=m, r=1, act=act, skew="none", flip_frac=0.05)
    L = W.layer_inputs(s, 31)
    idx = TB.recorded_route(L, s, 31)
    y, g = TR.run_replay(TR.dev_layer(L, act), idx, renorm=renorm)
    y_ref, g_ref = O.replay_forward(L["x"], idx, L["W_r"], L["beta"], L["W_gate"], L["W_up"],
                                    L["W_down"], renorm)
    compare_gates(g, g_ref, "tile")
    compare_rows(y, y_ref, act, "tile")
    dy = W.upstream_grad(s, 31)
    grads = TB.run_bwd(L, idx, dy, act, renorm=renorm)
    ref = TB.oracle_bwd(L, idx, dy, renorm)
    # renormalised weights of one route per token have no router gradient (g = 1)
    names = [n for n in TB.GRADS if not (k == 1 and renorm and n in ("dW_r", "dbeta"))]
    TB.compare(grads, ref, act, str(case), names)
    if k == 1 and renorm:
        assert np.all(grads["dW_r"] == 0.0) and np.all(grads["dbeta"] == 0.0)
    TS.run_pair(L, s, idx, dy, renorm)
