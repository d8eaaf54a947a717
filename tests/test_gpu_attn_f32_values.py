"""fp32 attention away from small, finite scores: what the values of q, k and v may do to a result."""
import pytest
import torch

from tests.gpu_util import print_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import paper_2605_23163_amd as F
    F.load_library()
    return F


def test_rows_of_block_keys_two_gigabytes_apart(F):
    # heads so many that the 16 keys of a tile span more than 2^31 bytes (15 x 580 000 heads x 64 x 4): every key must
    # count.  Checked against the same problem cut down to a few heads.
    B, Hkv, D = 16, 580000, 64
    print_case(test="wide_rows", Hkv=Hkv)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, bk, bv = (torch.randn((1, B, Hkv, D), device="cuda", generator=g) for _ in range(3))
    none = torch.empty((0, Hkv, D), device="cuda")
    out = F.fdd_block_attn(q, none, none, bk, bv)
    heads = torch.tensor([0, 1, 290000, Hkv - 1], device="cuda")
    cut = [x[:, :, heads].contiguous() for x in (q, bk, bv)]
    small = F.fdd_block_attn(cut[0], none[:, :4].contiguous(), none[:, :4].contiguous(), cut[1], cut[2])
    torch.cuda.synchronize()
    assert (out[:, :, heads] - small).abs().max().item() <= 1e-5
