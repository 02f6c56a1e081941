"""The fp64 vector router adds a logit's terms in K order, whatever the batch, the
number of columns or the kernel form: a token's logits do not depend on what else is
in the call.  The inputs make the order visible after the rounding to fp32: terms of
about 2^80 that cancel exactly, with terms of order one between them, some of which a
partial sum absorbs.  Products of two fp32 (or bf16) values are exact in fp64, so
the reference is the plain serial loop, bit for bit."""
import numpy as np
import pytest

import workloads as W
from tests.parity import to_dev

pytestmark = pytest.mark.gpu

CASES = [
    # (d, N, r, act): one and two columns per thread, odd column counts, ends of K steps, the
    # forms for up to and above 64 columns
    (64, 8, 0, "f32"), (64, 8, 4, "f32"), (61, 5, 2, "f32"), (132, 32, 1, "f32"), (260, 61, 3, "f32"),
    (128, 64, 0, "f32"), (68, 64, 8, "f32"), (100, 33, 0, "bf16"), (76, 48, 16, "bf16"),
]
SIZES = (1, 7, 40, 4097, 9000)


def problem(d, N, r, act, T):
    rng = np.random.default_rng([d, N, r])
    x = rng.uniform(0.5, 1.0, (T, d))
    w = rng.uniform(-1.0, 1.0, (d, N + r))
    for k in range(0, d - 2, 4):
        x[:, k] *= 2.0 ** 80
        if act == "bf16":
            x[:, k] = W.round_to_bf16(x[:, k].astype(np.float32))
        x[:, k + 2] = -x[:, k]
        w[k + 2] = w[k]
    x = x.astype(np.float32)
    if act == "bf16":
        x = W.round_to_bf16(x)
    return x, w.astype(np.float32)


@pytest.mark.parametrize("case", CASES, ids=["d%d_N%d_r%d_%s" % c for c in CASES])
def test_logits_are_the_serial_sum(case):
    import torch
    from paper_2606_00395_amd import binding as B
    d, N, r, act = case
    x, w = problem(d, N, r, act, max(SIZES))
    ref = np.zeros((len(x), N))
    for k in range(d):
        ref += x[:, k:k + 1].astype(np.float64) * w[k, :N].astype(np.float64)
    ref = ref.astype(np.float32)
    assert np.isfinite(ref).all()
    W_r = to_dev(w[:, :N])
    A = to_dev(w[:, N:]) if r else None
    Bf = torch.zeros((r, N), device="cuda") if r else None
    for T in SIZES:
        p = torch.empty((T, N), device="cuda")
        ids = torch.empty((T, 1), dtype=torch.int32, device="cuda")
        B.route_predict(to_dev(x[:T], act), W_r, None, A, Bf, 1, ids, logits_out=p)
        np.testing.assert_array_equal(p.cpu().numpy(), ref[:T], err_msg=f"first {T} tokens")
        np.testing.assert_array_equal(ids[:, 0].cpu().numpy(), ref[:T].argmax(1))
