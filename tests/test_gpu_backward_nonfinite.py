"""Replay backward of an upstream gradient with one infinity, in the last route of an
expert: the padding of that expert's last K step must not touch it.  dW_down[e] =
sum_q dy_q^T (g_q H_q), so row c of it is the infinity times g_q H_q, an infinity of that
value's sign, and every other row stays finite and unchanged.  g_q H_q itself comes from a
pass whose dy is one at that place and zero elsewhere."""
import numpy as np
import pytest

import workloads as W
from tests import test_gpu_backward as TB

pytestmark = pytest.mark.gpu

COUNTS = (1, 5, 31, 32, 33, 64, 100, 129)


@pytest.mark.parametrize("d,m,act", [(256, 256, "bf16"), (512, 384, "bf16"), (96, 40, "bf16"), (40, 72, "f32")],
                         ids=["mfma", "half_panel", "tile_bf16", "tile_fp32"])
@pytest.mark.parametrize("value", [np.inf, -np.inf], ids=["inf", "minus_inf"])
def test_infinity_in_an_experts_last_route(d, m, act, value):
    T, N, col = sum(COUNTS), len(COUNTS), 3
    s = W.LayerShape("nonfinite", T=T, d=d, N=N, k=1, m=m, r=0, act=act, skew="none")
    L = W.layer_inputs(s, 43)
    idx = np.random.default_rng(43).permutation(np.repeat(np.arange(N), COUNTS)).reshape(T, 1)
    last = [int(np.flatnonzero(idx[:, 0] == e)[-1]) for e in range(N)]
    dy = W.upstream_grad(s, 43)
    one = np.zeros_like(dy)
    one[last, col] = 1.0
    gH = TB.run_bwd(L, idx, one, act, renorm=False)["dW_down"][:, col]
    clean = TB.run_bwd(L, idx, dy, act, renorm=False)["dW_down"]
    dy[last, col] = value
    got = TB.run_bwd(L, idx, dy, act, renorm=False)["dW_down"]
    assert np.mean(gH != 0.0) > 0.9
    with np.errstate(invalid="ignore"):
        want = value * np.sign(gH)
    np.testing.assert_array_equal(got[:, col], want)
    rest = np.arange(d) != col
    np.testing.assert_array_equal(got[:, rest], clean[:, rest])
