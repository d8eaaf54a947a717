"""Calls on a stream that is not torch's current one: memory that the binding allocates belongs to the call's stream."""
import ctypes as C

import pytest
import torch

from tests.gpu_util import print_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import paper_2605_23163_amd as F
    F.load_library()
    return F


class Spy:
    """The library with the parameters of every call kept."""

    def __init__(self, lib):
        self.lib, self.seen = lib, []

    def __getattr__(self, name):
        fn = getattr(self.lib, name)

        def call(*a):
            if a and hasattr(a[0], "_obj"):
                p = type(a[0]._obj)()
                C.pointer(p)[0] = a[0]._obj
                self.seen.append((name, p))
            return fn(*a)
        return call


def calls(F):
    dev = "cuda"
    q = torch.randn(1, 8, 4, 64, device=dev)
    pk, pv = torch.randn(300, 1, 64, device=dev), torch.randn(300, 1, 64, device=dev)
    bk, bv = torch.randn(1, 8, 1, 64, device=dev), torch.randn(1, 8, 1, 64, device=dev)
    x = torch.randn(2, 8, 5000, device=dev)
    mask = torch.ones(2, 8, dtype=torch.uint8, device=dev)
    tok, drafts = (torch.zeros(2, 8, dtype=torch.int32, device=dev) for _ in range(2))
    pv16 = pv.to(torch.bfloat16)
    return {
        "fdd_block_attn": lambda **k: F.fdd_block_attn(q, pk, pv, bk, bv, splits=2, **k),
        "fdd_block_attn_batched": lambda **k: F.fdd_block_attn_batched(q[None], pk[None], pv[None], bk[None], bv[None], splits=2, **k),
        "fdd_unmask_step": lambda **k: F.fdd_unmask_step(x, mask, None, 0.9, tok, **k)[1:],
        "fdd_verify_step": lambda **k: F.fdd_verify_step(x, mask, None, drafts, tok, **k)[1:],
        "fdd_prefix_pack": lambda **k: F.fdd_prefix_pack(pv16, **k),
        "fdd_fork_block": lambda **k: F.fdd_fork_block(bk, 3, **k),
        "fdd_traj_mean": lambda **k: F.fdd_traj_mean(q[0], **k),
    }


class Handle:
    """Any object with a stream's handle is taken for the stream."""

    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


@pytest.mark.parametrize("wrap", [lambda s: s, Handle])
@pytest.mark.parametrize("name", ["fdd_block_attn", "fdd_block_attn_batched", "fdd_unmask_step", "fdd_verify_step"])
def test_scratch_is_not_handed_to_the_current_stream(F, monkeypatch, name, wrap):
    from paper_2605_23163_amd import binding
    print_case(test="scratch_stream", name=name)
    spy = Spy(binding.load_library())
    monkeypatch.setattr(binding, "_lib", spy)
    call = calls(F)[name]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    kept = call(stream=wrap(s))
    p = [p for n, p in spy.seen if not n.endswith("_workspace")][-1]
    assert p.stream == s.cuda_stream and p.workspace_bytes > 0
    # the call may still run on s: what is allocated for the current stream now must not be its scratch
    fresh = [torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda") for _ in range(4)]
    assert all(t.data_ptr() + t.numel() <= p.workspace or p.workspace + p.workspace_bytes <= t.data_ptr() for t in fresh)
    torch.cuda.synchronize()
    del kept


@pytest.mark.parametrize("name", ["fdd_block_attn", "fdd_block_attn_batched", "fdd_unmask_step", "fdd_verify_step", "fdd_prefix_pack",
                                  "fdd_fork_block", "fdd_traj_mean"])
def test_outputs_do_not_take_memory_in_use(F, name):
    print_case(test="output_stream", name=name)
    call = calls(F)[name]
    s = torch.cuda.Stream()
    tensors = lambda r: [r] if isinstance(r, torch.Tensor) else list(r)
    sizes = [t.numel() * t.element_size() for t in tensors(call())]
    torch.cuda.synchronize()
    # memory that work on the current stream still uses after its tensor is gone
    busy = [torch.empty(n, dtype=torch.uint8, device="cuda") for n in sizes for _ in range(3)]
    spans = [(t.data_ptr(), t.data_ptr() + t.numel()) for t in busy]
    inputs_ready = torch.cuda.Event()
    inputs_ready.record()
    torch.cuda._sleep(20_000_000)
    for t in busy:
        t.fill_(7)
    del busy, t
    s.wait_event(inputs_ready)
    res = tensors(call(stream=s))
    for t in res:
        lo, hi = t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()
        assert all(hi <= a or b <= lo for a, b in spans), "an output lies in memory that the current stream is writing"
    # and memory of an output that the current stream reads is not reused by a later call on s
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda._sleep(20_000_000)
    copies = [t.clone() for t in res]
    spans = [(t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in res]
    del res, t
    again = tensors(call(stream=s))
    for t in again:
        lo, hi = t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()
        assert all(hi <= a or b <= lo for a, b in spans), "an output lies in memory that the current stream is reading"
    torch.cuda.synchronize()
    del copies
