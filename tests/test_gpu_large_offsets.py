"""Activations of nearly 2^31 elements: the expert GEMMs copy rows at 32-bit byte offsets
from the tensor's start, up to the last below 4 GiB.  The last tokens of such a batch must
come out as from a batch of these tokens alone: outputs, weights and input gradients bitwise;
weight gradients, with the upstream gradient zero before them, up to the order of fp32 sums
(300 routes: 300 * 2^-24 of the sum of magnitudes at most, a few 1e-6 relative)."""
import pytest

pytestmark = pytest.mark.gpu


def test_rows_near_4_gib():
    import torch
    from paper_2606_00395_amd import binding as B
    T, d, N, m, tail = 520000, 4096, 4, 128, 300
    assert 2 ** 32 - 2 ** 27 < 2 * T * d < 2 ** 32
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(47)

    def randn(*shape, std=1.0, dt=torch.bfloat16):
        return torch.randn(shape, generator=g, device="cuda").mul_(std).to(dt)

    x = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 65000):
        x[t:t + 65000] = randn(65000, d)
    dy = torch.zeros_like(x)
    dy[-tail:] = randn(tail, d)
    idx = torch.randint(0, N, (T, 1), generator=g, device="cuda", dtype=torch.int32)
    W_r, b_r = randn(d, N, std=0.02, dt=torch.float32), randn(N, dt=torch.float32)
    W = [randn(N, m, d, std=0.02), randn(N, m, d, std=0.02), randn(N, d, m, std=0.02)]

    def layer(x, idx, dy):
        y, gate = torch.empty_like(x), torch.empty(idx.shape, device="cuda")
        B.moe_replay_forward(x, idx, W_r, b_r, *W, y, gate_out=gate, renorm=False)
        grads = [torch.empty_like(x), torch.empty_like(W_r), torch.empty_like(b_r)]
        grads += [torch.empty(w.shape, device="cuda") for w in W]
        B.moe_replay_backward(x, idx, W_r, b_r, *W, dy, *grads, renorm=False)
        torch.cuda.synchronize()
        return [y[-tail:], gate[-tail:], grads[0][-tail:]], grads[3:]

    rows, weights = layer(x, idx, dy)
    rows1, weights1 = layer(x[-tail:].contiguous(), idx[-tail:].contiguous(), dy[-tail:].contiguous())
    for a, b, n in zip(rows, rows1, ("y", "gate", "dx")):
        assert torch.equal(a, b), n
    for a, b, n in zip(weights, weights1, ("dW_gate", "dW_up", "dW_down")):
        assert b.norm() > 0 and (a - b).norm() <= 1e-5 * b.norm(), n
