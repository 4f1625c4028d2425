"""hilore_dequant_lora_grad over the row-block counts of one pass (R = 2, 3, 4 and
their remainders), at the edges of its strips and k-steps.

Integer-valued operands: every partial sum is an integer below 2^24, so fp32
accumulation is exact in any order and the result must equal the fp64 product.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def operands(K, M, r, code, block):
    g = torch.Generator(device="cuda").manual_seed(1000 * r + K + M)
    x = torch.randint(-7, 8, (K, M), generator=g, device="cuda").float()
    dh = torch.randint(-8, 9, (K, r), generator=g, device="cuda").to(torch.bfloat16)
    if block:  # a power-of-two scale per block
        e = torch.randint(-2, 3, (K, M // block), generator=g, device="cuda")
        scales = torch.exp2(e.float())
    if code == 0:
        codes = (x.to(torch.int8) * 16).view(torch.uint8)
        scales = scales / 16
        xhat = x * (scales * 16).repeat_interleave(block, 1)
    else:
        codes = x.to(torch.float8_e4m3fn).view(torch.uint8)
        xhat = x * scales.repeat_interleave(block, 1) if block else x
        scales = scales if block else None
    return codes, scales, dh, xhat


@pytest.mark.parametrize("r", [18, 32, 40, 48, 50, 64])
@pytest.mark.parametrize("code,block,K,M", [
    (2, 0, 1, 16),        # one token, one column group
    (2, 0, 33, 144),      # a second k-step of one token; one slab and a bit
    (0, 32, 129, 288),    # the second strip's first slab, 32 columns of it
    (1, 32, 1000, 416),   # a strip and 160 columns
    (0, 64, 4097, 896),   # narrow unit: equal parts per strip, a last token alone
    (1, 128, 515, 3584),  # 14 strips
    (0, 256, 97, 8448),   # 33 strips: consecutive ranges per XCD, ranges across strips
])
def test_integer_exact(hl, code, block, K, M, r):
    codes, scales, dh, xhat = operands(K, M, r, code, block)
    da = torch.full((r, M), float("nan"), device="cuda")
    ws = torch.full((hl.hilore_lora_grad_workspace_bytes(K, M, r) // 4,), float("nan"), device="cuda")
    hl.hilore_dequant_lora_grad(codes, scales, code, block, dh, da, K, M, r, 2.0, False, ws)
    want = 2.0 * (dh.double().t().contiguous() @ xhat.double())
    assert torch.equal(da.double(), want)
    hl.hilore_dequant_lora_grad(codes, scales, code, block, dh, da, K, M, r, 2.0, True, ws)
    assert torch.equal(da.double(), 2 * want)


@pytest.mark.parametrize("r", [34, 48, 64, 80])
@pytest.mark.parametrize("code,block,K,M", [
    (1, 128, 2049, 1152),   # 5 strips: ranges of 8 k-steps
    (0, 64, 8200, 1152),    # ranges of 16, an odd number of k-steps
    (2, 0, 16385, 272),     # 2 strips, 33 parts each
    (0, 32, 160, 8192),     # 32 strips, one k-step or none a workgroup: cooperative to 64 rows
    (1, 64, 1400, 9728),    # 38 strips, ranges across strips, cooperative
    (1, 128, 4099, 8448),   # 33 strips, ranges across strips, slab
    (0, 256, 1500, 16384),  # 64 strips of four ranges each, slab
])
def test_splits(hl, code, block, K, M, r):
    """Both kernels of 33 to 64 rows and every rule of the split, no more workspace than asked."""
    test_integer_exact(hl, code, block, K, M, r)
