"""Helpers for the GPU parity tests: host arrays <-> device tensors."""
import numpy as np
import torch

import fdd_workloads as W


def to_dev(a, dtype=None):
    """numpy array in storage type (uint16 = bf16 bits) -> cuda tensor."""
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    return torch.from_numpy(a).cuda()


def to_f64(t):
    """cuda tensor -> float64 numpy (exact widening)."""
    return t.detach().to(torch.float64).cpu().numpy()


def storage(x, dtype):
    return W.to_storage(np.asarray(x, dtype=np.float32), dtype)


def rand_attn(rng, N, B, L, Hq, Hkv, D, dtype, std=1.0):
    f = lambda *s: storage(rng.standard_normal(s) * std, dtype)
    return dict(q=f(N, B, Hq, D), prefix_k=f(L, Hkv, D), prefix_v=f(L, Hkv, D),
                block_k=f(N, B, Hkv, D), block_v=f(N, B, Hkv, D))


def row_error(out, ref):
    """Largest error of an output row (last axis) in norm, relative to the row.  Three roundings to bf16 (probabilities, segments'
    averages, outputs), each of 2^-9 to 2^-8 of a value, leave 3e-3 of it whatever the number of keys; ROW_TOL is five times
    that, and less than what a tile of 64 keys too few leaves among 20000 (6e-2 and more)."""
    return float((np.linalg.norm(out - ref, axis=-1) / np.linalg.norm(ref, axis=-1)).max())


ROW_TOL = 1.5e-2


def print_case(**kw):
    print("[case]", " ".join(f"{k}={v}" for k, v in kw.items()), flush=True)
