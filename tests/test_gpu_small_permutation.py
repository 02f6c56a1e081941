"""The one-workgroup permutation of small batches (at most 16384 routes) against
the three-launch one: a batch's rows must be bitwise those of the same tokens at
the head of a batch that is over the limit, out-of-range ids (which are skipped)
included.  Parity with the oracle is tests/test_gpu_replay.py's."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_replay import dev_layer, run_replay

pytestmark = pytest.mark.gpu

LIMIT = 16384
CASES = [
    # (N, k, act, d, m, batch sizes): edges of 64 routes, 1024 a pass, the limit
    (8, 2, "f32", 24, 16, (1, 31, 32, 33, 511, 512, 513, 4097, 8191, 8192)),
    (1024, 7, "f32", 24, 16, (1, 9, 10, 147, 586, 2340)),
    (64, 8, "bf16", 256, 128, (1, 8, 129, 1024, 2047, 2048)),
    (1, 1, "f32", 24, 16, (64, 1025, LIMIT)),
]


@pytest.mark.parametrize("bad_ids", [False, True], ids=["valid", "some_out_of_range"])
@pytest.mark.parametrize("case", CASES, ids=[f"N{c[0]}_k{c[1]}_{c[2]}" for c in CASES])
def test_small_batches_match_a_large_one(case, bad_ids):
    N, k, act, d, m, sizes = case
    T = LIMIT // k + 100
    s = W.LayerShape("perm", T=T, d=d, N=N, k=k, m=m, r=0, act=act, skew="none")
    L = W.layer_inputs(s, 29)
    rng = np.random.default_rng(29)
    idx = np.argsort(rng.random((T, N)), axis=1)[:, :k].astype(np.int32)
    if bad_ids:
        idx[rng.random((T, k)) < 0.1] = -3
        idx[rng.random((T, k)) < 0.1] = N
    D = dev_layer(L, act)
    y, g = run_replay(D, idx, idx_dtype="int16", ldi_pad=1)
    for t in sizes:
        ys, gs = run_replay(D, idx[:t], ldi_pad=t % 2, x=D["x"][:t])
        np.testing.assert_array_equal(gs, g[:t], err_msg=f"weights of the first {t} tokens")
        np.testing.assert_array_equal(ys, y[:t], err_msg=f"outputs of the first {t} tokens")
