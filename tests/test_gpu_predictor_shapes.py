"""The predictor loss's three-launch form (bf16, rank <= 64, at most 192 experts, d a
multiple of 64) at the edges of its 8-token workgroups, 16-column rank tiles,
64-expert groups and token slices, and just outside it, against the oracle
(bar: Frobenius ratio <= 1e-5, as tests/test_gpu_predictor.py)."""
import pytest

from oracle import pr2_oracle as O
import workloads as W
from tests import test_gpu_predictor as TP
from tests.parity import to_dev

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


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_operands_at_any_4_byte_address(shift):
    """A, B, the router, its bias and p_old may be views into a larger buffer that
    start at any float: the same bits as from fresh tensors."""
    import torch
    from paper_2606_00395_amd import binding as B
    s = W.LayerShape("pred", T=65, d=256, N=64, k=1, m=8, r=16, act="bf16", skew="hot8")
    L = W.layer_inputs(s, 37, experts=False)
    x = to_dev(L["x"], "bf16")
    ops = {n: to_dev(L[n]) for n in ("W_r", "beta", "A", "B")}
    ops["p_old"] = to_dev(O.router_logits(L["x"], L["W_r"], L["beta"]).astype("float32") + 0.1 * L["x"][:, :64])

    def loss(off):
        t = {}
        for n, v in ops.items():
            flat = torch.empty(v.numel() + off, device="cuda")
            t[n] = flat[off:].view(v.shape)
            t[n].copy_(v)
            assert t[n].data_ptr() % 16 == 4 * off
        out = [torch.empty(n, device="cuda") for n in ((1,), (s.d, s.r), (s.r, s.N), (s.T,))]
        B.predictor_loss(x, t["W_r"], t["beta"], x, t["p_old"], t["A"], t["B"], *out)
        torch.cuda.synchronize()
        return out

    for a, b in zip(loss(shift), loss(0)):
        assert torch.equal(a, b) and torch.isfinite(a).all()
