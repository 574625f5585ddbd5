"""Very small and very large gradients through every way that a block above 128 x 128 takes (bf16 or float32 gradients, 16-byte aligned
or not, filtered or not), against float64: products that split their operands on the way into LDS scale them by the block's largest
element, products on planes by scales of their own."""
import numpy as np
import pytest

from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma", [1e-15, 1e13])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("beta1", [0.0, 0.9])
@pytest.mark.parametrize("bf16", [False, True])
def test_factors_and_direction(bf16, beta1, skew, sigma):
    import torch
    m, n = 264, 136
    gen = torch.Generator(device="cuda")
    gen.manual_seed(29)
    dtype = torch.bfloat16 if bf16 else torch.float32
    opt = B.Shampoo([(m, n)], 512, 0.99, 1e-6 * sigma * sigma, 0.25, 1, 0, grad_dtype=B.GRAD_BF16 if bf16 else B.GRAD_F32, beta1=beta1)
    w = [torch.zeros(m, n, device="cuda")]
    beta, b1 = float(np.float32(0.99)), float(np.float32(beta1))
    L = R = Gf = 0.0
    for t in range(3):
        g = torch.empty(m * n + 8, device="cuda", dtype=dtype)[skew:skew + m * n].view(m, n)
        g.copy_(torch.randn(m, n, device="cuda", generator=gen) * sigma)
        opt.step(w, [g], 0.01, t)
        x = g.double()
        L, R, Gf = beta * L + (1 - beta) * (x @ x.T), beta * R + (1 - beta) * (x.T @ x), b1 * Gf + (1 - b1) * x
    get = lambda which: opt.get(0, 0, which).double()
    P = get(B.GET_LINV) @ Gf @ get(B.GET_RINV)
    off = [float((get(which) - x).norm() / x.norm()) for which, x in ((B.GET_L, L), (B.GET_R, R), (B.GET_PSH, P))]
    print("    L %.1e R %.1e P %.1e" % tuple(off), flush=True)
    # factors: three roundings to float32, 6e-8 each, and (bf16) float32 sums over up to 264 values of k, 6e-8 sqrt(264 / 16) at random;
    # direction: two such sums, the filter's roundings, and 2^-22 of an element in two fp16 planes
    assert off[0] <= 4.2e-7 and off[1] <= 4.2e-7 and off[2] <= 1.5e-6, off
