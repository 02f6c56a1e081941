"""The predictor loss's three-launch form (bf16, rank <= 64, at most 192 experts, d a
multiple of 64) at the edges of its 8-token workgroups, 16-column rank tiles,
64-expert groups and token slices, and just outside it, against the oracle
(bar: Frobenius ratio <= 1e-5, as tests/test_gpu_predictor.py)."""
import pytest

import workloads as W
from tests import test_gpu_predictor as TP

pytestmark = pytest.mark.gpu

CASES = [
    # (T, d, N, r, kind)
    (1, 64, 2, 1, 0), (7, 128, 5, 3, 1), (8, 64, 64, 16, 0), (9, 192, 65, 17, 1),
    (63, 512, 128, 32, 0), (65, 256, 129, 33, 0), (257, 320, 192, 64, 1),
    (4097, 128, 24, 5, 0),                      # 64 slices of 65 tokens
    (100, 96, 32, 8, 0), (100, 128, 193, 8, 0), (100, 128, 32, 65, 1),   # other forms
]


@pytest.mark.parametrize("case", CASES, ids=["T%d_d%d_N%d_r%d_kind%d" % c for c in CASES])
def test_predictor_shapes(case):
    T, d, N, r, kind = case
    s = W.LayerShape("pred", T=T, d=d, N=N, k=1, m=8, r=r, act="bf16", skew="none")
    L = W.layer_inputs(s, 37, experts=False)
    g, (kl_ref, dA_ref, dB_ref) = TP.run_loss(L, s, T, kind)
    errs = {"kl": TP.frob(g["kl"], kl_ref), "loss": abs(g["loss"] - kl_ref.mean()) / kl_ref.mean(),
            "dA": TP.frob(g["dA"], dA_ref), "dB": TP.frob(g["dB"], dB_ref)}
    assert max(errs.values()) <= TP.RTOL, errs
