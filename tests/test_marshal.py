"""Native argument marshalling: the structs are those that binding.py fills in Python, byte for byte, and whatever is not
the ordinary case is left to Python, whose checks then accept it or raise."""
import ctypes as C

import pytest
import torch

from paper_2605_23163_amd import binding as Bd


@pytest.fixture(scope="module")
def M():
    Bd.load_library()
    if Bd._marshal is None:
        pytest.skip("built without torch's headers")
    return Bd._marshal


def attn_args(dev, N=2, B=3, L=70, Hq=4, Hkv=2, D=64, dtype=torch.bfloat16, ext=False, **kw):
    z = lambda *s: torch.zeros(s, dtype=dtype, device=dev)
    a = dict(q=z(N, B, Hq, D), prefix_k=z(L, Hkv, D), prefix_v=z(L, Hkv, D), block_k=z(N, B, Hkv, D), block_v=z(N, B, Hkv, D),
             scaffold_mask=None, out=z(N, B, Hq, D), prefix_v_packed=None, ext_k=None, ext_v=None, q_positions=None, E=0,
             causal_block=False, splits=0, scale=None)
    if ext:
        a.update(ext_k=z(N, 9, Hkv, D), ext_v=z(N, 9, Hkv, D), E=5)
    a.update(kw)
    return a


def native(M, a):
    p = Bd.AttnParams()
    return M.attn(C.addressof(p), *a.values()), p


def unmask_args(dev, N=2, B=5, V=33, dtype=torch.float32, refresh=False, **kw):
    e = lambda s, t: torch.zeros(s, dtype=t, device=dev)
    a = dict(logits=e((N, B, V), dtype), mask=e((N, B), torch.uint8), scaffold_mask=e((N, B), torch.uint8), tokens=e((N, B), torch.int32),
             confidences=e((N, B), torch.float32), n_unmasked=e((N,), torch.int32), committed=e((N, B), torch.uint8), tau=0.9, refresh=None)
    if refresh:
        k = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device=dev)
        a["refresh"] = (k(7, 2, 64), k(7, 2, 64), k(N, B, 2, 64), k(N, B, 2, 64))
    a.update(kw)
    return a


def test_cpu_tensors_are_left_to_python(M):
    assert native(M, attn_args("cpu"))[0] is False
    p = Bd.UnmaskParams()
    assert M.unmask(C.addressof(p), *unmask_args("cpu").values()) is False
    with pytest.raises(ValueError, match="GPU memory"):
        a = attn_args("cpu")
        Bd.fdd_block_attn(**a)
    with pytest.raises(TypeError):
        M.attn(C.addressof(p), 1)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(), dict(dtype=torch.float32, L=0), dict(ext=True, causal_block=True), dict(splits=3, scale=0.25), dict(scale=2)])
def test_attention_struct(M, kw):
    a = attn_args("cuda", **kw)
    a["scaffold_mask"] = torch.zeros(2, 3, dtype=torch.uint8, device="cuda")
    ok, p = native(M, a)
    r = Bd._attn_params(a["q"], a["prefix_k"], a["prefix_v"], a["block_k"], a["block_v"], a["scaffold_mask"], a["out"], a["scale"],
                        a["splits"], a["prefix_v_packed"], a["causal_block"], a["ext_k"], a["ext_v"], a["E"])
    assert ok is True and bytes(p) == bytes(r)
    qp = torch.arange(4, dtype=torch.int32, device="cuda")
    ok, p = native(M, dict(a, q_positions=qp))
    r.q_positions, r.n_q_positions = qp.data_ptr(), 4
    assert ok is True and bytes(p) == bytes(r)


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(), dict(dtype=torch.bfloat16, refresh=True), dict(scaffold_mask=None, tau=1)])
def test_unmask_struct(M, kw):
    a = unmask_args("cuda", **kw)
    p = Bd.UnmaskParams()
    assert M.unmask(C.addressof(p), *a.values()) is True
    r = Bd._unmask_params(a["logits"], a["mask"], a["scaffold_mask"], a["tokens"], a["tau"], a["confidences"], a["n_unmasked"], a["committed"], a["refresh"])
    assert bytes(p) == bytes(r)


@pytest.mark.gpu
def test_other_cases_are_left_to_python(M):
    a = attn_args("cuda")
    t = a["q"]

    class Sub(torch.Tensor):
        pass

    others = [dict(q=t[0]), dict(q=t.float()), dict(q=t.transpose(0, 1)), dict(out=t.transpose(2, 3)), dict(block_k=a["block_k"][:, :2]),
              dict(prefix_v=a["prefix_v"][:60]), dict(ext_k=t, ext_v=t, E=1), dict(E=1.0), dict(splits="a"), dict(scale="a"), dict(splits=2**40),
              dict(q_positions=torch.zeros(3, device="cuda")), dict(q=t.as_subclass(Sub)), dict(q=t.half()), dict(out=t.cpu()), dict(q=None)]
    for kw in others:
        assert native(M, dict(a, **kw))[0] is False, kw
    vmapped = []
    torch.func.vmap(lambda x: (vmapped.append(native(M, dict(a, q=x))[0]), x)[1])(torch.stack([t, t]))
    assert vmapped == [False]
    with torch.overrides.TorchFunctionMode():
        assert native(M, a)[0] is False
    u = unmask_args("cuda")
    for kw in (dict(mask=u["mask"].int()), dict(tokens=u["tokens"][:1]), dict(logits=u["logits"][0]), dict(refresh=(t, t)), dict(tau=None), dict(mask=u["mask"].cpu())):
        p = Bd.UnmaskParams()
        assert M.unmask(C.addressof(p), *dict(u, **kw).values()) is False, kw
    with pytest.raises(TypeError):
        Bd.fdd_unmask_step(**dict(u, mask=u["mask"].int()))
    with pytest.raises(ValueError):
        Bd.fdd_block_attn(**dict(a, q_positions=torch.zeros(3, device="cuda")))


def test_forks_of_cpu_tensors_are_left_to_python(M):
    assert M.fork(torch.zeros(4), 2, torch.zeros(2, 4)) is None
    with pytest.raises(ValueError, match="GPU memory"):
        Bd.fdd_fork_block(torch.zeros(4), 2, dst=torch.zeros(2, 4))
    with pytest.raises(TypeError):
        M.fork(torch.zeros(4), 2)


@pytest.mark.gpu
def test_fork_arguments(M):
    src = torch.zeros(3, 8, dtype=torch.bfloat16, device="cuda")
    for dst in (src.new_zeros(5, 3, 8), src.new_zeros(120), torch.zeros(5, 12, dtype=torch.int32, device="cuda")):
        assert M.fork(src, 5, dst) == (48, src.data_ptr(), dst.data_ptr())
    dst = src.new_zeros(5, 3, 8)
    others = [(src, 4, dst), (src, 0, dst), (src, -5, dst), (src, 5.0, dst), (src, 5, dst.cpu()), (src.t(), 5, dst), (src, 5, dst.transpose(0, 1)),
              (src, 5, None), (src.half()[:2], 5, dst), (src, 2**40, dst)]
    for a in others:
        assert M.fork(*a) is None, a[1]
    with torch.overrides.TorchFunctionMode():
        assert M.fork(src, 5, dst) is None
    with pytest.raises(ValueError):
        Bd.fdd_fork_block(src, 4, dst=dst)
