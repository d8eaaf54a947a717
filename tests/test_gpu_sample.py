"""The sampled verifier drops entries by an upper bound of their key: the tokens must be the oracle's all the same."""
import numpy as np
import pytest
import torch

import fdd_workloads as W
from tests.gpu_util import print_case, to_dev


@pytest.fixture(scope="module")
def F():
    import paper_2605_23163_amd as f
    f.load_library()
    return f


def test_noise_bound_is_never_below_the_noise(oracle):
    # the kernel's bound (float arithmetic as there, its fused multiply-add in 64 bits and rounded) against the
    # definition, for every value of the 23 bits the noise is made from
    k = np.arange(1 << 23, dtype=np.uint32)
    u = ((k.astype(np.float32) + np.float32(0.5)) * np.float32(2.0 ** -23)).astype(np.float32)
    noise = -oracle.flog2(-oracle.flog2(u))
    w = ((~(k << np.uint32(9)) >> np.uint32(9)).astype(np.float32) + np.float32(0.5)).astype(np.float32)
    bound = (w.view(np.uint32).astype(np.float32).astype(np.float64) * -2.0 ** -23 + np.float64(np.float32(149.47223))).astype(np.float32)
    assert np.all(bound - noise > 5e-4) and bound.max() <= np.float32(23.47223)
    for above, excess in ((0.5, 0.48), (0.875, 0.16), (0.99, 0.092)):   # and close where an entry can win
        assert np.all(bound[u > above] - noise[u > above] < excess)


# one position per block, so that the token of every row is seen.  V: one entry, less than a vector, rows that start at
# every place of a vector and of a generator block, several pieces; more than 1024 pieces and fewer, of 16 KB and less, around
# 256 of them (where a row is cut twice as often)
@pytest.mark.gpu
@pytest.mark.parametrize("case", [(1100, 1003, W.BF16, 0.7), (1100, 257, W.F32, 1.0), (30, 1, W.BF16, 1.0), (30, 7, W.BF16, 0.5),
                                  (64, 20485, W.BF16, 1.0), (40, 70001, W.BF16, 0.7), (24, 33003, W.F32, 0.7), (16, 152064, W.BF16, 1.0),
                                  (200, 8192, W.BF16, 0.7), (256, 8191, W.BF16, 0.7), (257, 9973, W.BF16, 1.0), (31, 4099, W.F32, 1.0)])
@pytest.mark.parametrize("spike", [0.0, 25.0])
def test_sampled_tokens_with_and_without_a_clear_winner(F, oracle, case, spike):
    N, V, dtype, temperature = case
    print_case(test="sample_bound", case=case, spike=spike)
    rng = np.random.default_rng(V + int(spike))
    x = (rng.standard_normal((N, 1, V)) * 2).astype(np.float32)
    at = rng.integers(0, V, N)
    x[np.arange(N), 0, at] += spike
    x[N // 2, 0, rng.integers(0, V, max(1, V // 3))] = -np.inf        # banned tokens
    x[N // 2, 0, at[N // 2]] = 1.0
    logits = W.to_storage(x, dtype)
    mask = np.ones((N, 1), dtype=np.uint8)
    # drafts: the spike, some other token, no token at all
    draft = np.where(rng.random(N) < 0.6, at, rng.integers(-2, V + 2, N)).astype(np.int32)[:, None]
    tokens = np.full((N, 1), -7, dtype=np.int32)
    ref = oracle.verify_step(logits, mask, None, draft, tokens, temperature=temperature, seed=77)
    m, t = torch.from_numpy(mask.copy()).cuda(), torch.from_numpy(tokens.copy()).cuda()
    F.fdd_verify_step(to_dev(logits), m, None, torch.from_numpy(draft).cuda(), t, temperature=temperature, seed=77)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(t.cpu().numpy(), ref["tokens"])
