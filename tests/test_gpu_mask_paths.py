"""Masking of bf16 logits on both sides of the size up to which they are stored through the L2 cache (128 MB), and on
rows and base addresses of every alignment, against plain PyTorch on the same bits."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _masked(logits, cls_bits, c):
    allowed = (cls_bits[:, (c // 32).long()] >> (c % 32)) & 1
    return torch.where(allowed.bool(), logits, torch.full_like(logits, float("-inf")))


@pytest.mark.parametrize("B,V,stride,offset", [(511, 131_072, 131_072, 0), (512, 131_072, 131_072, 0),
                                               (513, 131_072, 131_072, 0), (7, 4_099, 4_104, 0), (7, 4_099, 4_104, 1),
                                               (7, 4_099, 4_099, 0), (5, 2_049, 2_050, 3), (3, 15, 16, 0)])
def test_store_paths(B, V, stride, offset):
    import paper_2605_29986_amd as lib
    print(f"case B={B} V={V} stride={stride} offset={offset}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B + V)
    C = 777
    flat = torch.randint(-2**15, 2**15, (B * stride + 8,), device="cuda", generator=gen).to(torch.int16)
    flat &= 0x7F7F  # finite values: compared as numbers below, as bits outside the rows
    before = flat.clone()
    logits = flat[offset:offset + B * stride].view(torch.bfloat16).view(B, stride)[:, :V]
    c = torch.randint(0, C, (V,), device="cuda", generator=gen).to(torch.int32)
    cls_bits = torch.randint(-2**31, 2**31, (B, (C + 31) // 32), device="cuda", generator=gen).to(torch.int32)
    want = _masked(logits, cls_bits, c)
    lib.cfgzip_apply_mask(logits, cls_bits, class_of_token=c, C=C)
    assert torch.equal(logits, want)
    # nothing outside the rows is touched
    outside = torch.ones_like(flat, dtype=torch.bool)
    outside[offset:offset + B * stride].view(B, stride)[:, :V] = False
    assert torch.equal(flat[outside], before[outside])
