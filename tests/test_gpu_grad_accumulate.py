"""Weight-gradient sums: dst = src and dst += src (bf16 into fp32), bitwise
equal to torch's conversion and addition (one fp32 rounding each), around a
workgroup's 2048 values; a size that is no multiple of 8 is refused."""
import pytest


def test_size_check():
    from paper_2606_01143_amd import binding as B
    f = B.lib().spr_grad_accumulate
    assert B.STATUS[f(12, 0x7F0000000000, 0x7F0000100000, 0, None)] == "SPR_ERR_INVALID_ARG"
    assert B.STATUS[f(16, 0x7F0000000000, 0x7F0000000010, 0, None)] == "SPR_ERR_ALIASING"


@pytest.mark.gpu
@pytest.mark.parametrize("n", [8, 2040, 2048, 2056, 3 * 2048 + 8, 1 << 20])
def test_grad_accumulate(gpu, n):
    import torch
    from paper_2606_01143_amd import binding as B
    print(f"[gpu-case] grad accumulate n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    src = torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    dst = torch.randn(n + 8, generator=g, device="cuda")
    want, tail = dst[:n] + src.float(), dst[n:].clone()
    B.grad_accumulate(dst[:n], src)
    assert torch.equal(dst[:n], want) and torch.equal(dst[n:], tail)
    B.grad_accumulate(dst[:n], src, overwrite=True)
    assert torch.equal(dst[:n], src.float()) and torch.equal(dst[n:], tail)
