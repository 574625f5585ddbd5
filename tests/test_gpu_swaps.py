"""The swap of a tensor block's first two indices (permute_12_kernel in csrc/tensor_blocks.h): widths of the last dimension on both sides of
every change of its tile and of the limit of 72, other dimensions that the tiles do not divide.  The swap only moves data, so the
factor of the middle dimension, formed from the swapped block, is held against float64."""
import pytest

from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("post", [2, 9, 10, 18, 19, 36, 37, 72, 73])
@pytest.mark.parametrize("shape,bf16", [((33, 17), False), ((35, 50), True)])
def test_factor_of_the_middle_dimension(shape, post, bf16):
    import torch
    shape = shape + (post,)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(shape))
    g = torch.randn(shape, device="cuda", generator=gen)
    if bf16:
        g = g.bfloat16()
    opt = B.Shampoo([shape], max(shape), 1.0, 1e-12, 0.25, 1 << 20, 1 << 20, grad_dtype=B.GRAD_BF16 if bf16 else B.GRAD_F32)
    opt.step([torch.zeros(shape, device="cuda")], [g], 0.01, 0)
    x = g.double()
    exact = torch.einsum("iaj,ibj->ab", x.cpu(), x.cpu())
    err = float((opt.get(0, 0, B.GET_L2).double().cpu() - exact).norm() / exact.norm())
    print(f"    {shape}: {err:.1e}", flush=True)
    # sums in float64, one rounding of the result: 2^-24; products of terms up to 2^-24 each
    assert err <= 2.4e-7, (shape, err)


@pytest.mark.parametrize("shape", [(40, 33, 40), (16, 9, 5, 24)])
def test_there_and_back(shape):
    """Wide last dimensions: the swap back is a launch of its own."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    opt = B.Shampoo([shape], max(shape), 0.99, 1e-12, 0.25, 1, 0)
    w = [torch.zeros(shape, device="cuda")]
    for t in range(2):
        g = torch.randn(shape, device="cuda", generator=gen)
        opt.step(w, [g], 0.01, t)
    x = g.double()
    for mode, root in enumerate([B.GET_LINV, B.GET_L2INV] + ([B.GET_L3INV] if len(shape) == 4 else []) + [B.GET_RINV]):
        x = torch.movedim(torch.tensordot(opt.get(0, 0, root).double(), x, dims=([1], [mode])), 0, mode)
    err = float((opt.get(0, 0, B.GET_PSH).double().reshape(shape) - x).norm() / x.norm())
    print(f"    {shape}: {err:.1e}", flush=True)
    assert err <= 1.4e-6, (shape, err)     # as in test_gpu_narrow_products.py
