"""Products of float32 operands in tiles of 128 x 128 and of 64 x 64 (csrc/gemm_mfma.h): few blocks take the small tile, many the
large one.  An element is the same sum in both, so both give the same bits; and those of float64."""
import numpy as np
import pytest

from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu


# one matrix and as many as exceed 1024 large tiles; sizes around the tiles' edges that no 16-byte load or plane divides
@pytest.mark.parametrize("m,n", [(129, 131), (191, 65), (130, 257), (67, 321), (3, 259), (255, 193)])
@pytest.mark.parametrize("grad,cores", [("f32", B.MATRIX_CORES_AUTO), ("bf16", B.MATRIX_CORES_AUTO), ("f32", B.MATRIX_CORES_FP32)])
def test_both_tiles(m, n, grad, cores):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m * n)
    dtype = torch.float32 if grad == "f32" else torch.bfloat16
    tiles = min(-(-m // 128) * -(-n // 128), *(t * (t + 1) // 2 for t in (-(-m // 128), -(-n // 128))))
    count = 1100 // tiles + 1
    few, many = (B.Shampoo([(m, n)] * c, 512, 0.99, 1e-6, 0.25, 1, 0, grad_dtype=B.GRAD_F32 if grad == "f32" else B.GRAD_BF16,
                           precond_matrix_cores=cores) for c in (1, count))
    w1, w2 = [torch.zeros(m, n, device="cuda")], [torch.zeros(m, n, device="cuda") for _ in range(count)]
    L = R = 0.0
    beta = float(np.float32(0.99))
    for t in range(2):
        g = (torch.randn(m, n, device="cuda", generator=gen) * 1e-2).to(dtype)
        few.step(w1, [g], 0.01, t)
        many.step(w2, [g.clone() if i in (0, count - 1) else torch.ones_like(g) for i in range(count)], 0.01, t)
        x = g.double()
        L, R = beta * L + (1 - beta) * (x @ x.T), beta * R + (1 - beta) * (x.T @ x)
    for which in (B.GET_L, B.GET_R, B.GET_PSH):
        a = few.get(0, 0, which)
        assert torch.equal(a, many.get(0, 0, which)) and torch.equal(a, many.get(count - 1, 0, which)), which
    get = lambda which: few.get(0, 0, which).double()
    P = get(B.GET_LINV) @ x @ get(B.GET_RINV)
    rel = lambda a, b: float((a - b).norm() / b.norm())
    # float32 storage of each of two steps; two float32 roundings per element of P beside sums over up to 321 values of k that
    # are rounded at 2^-24 of at most all of them (a random walk: sqrt(321) 6e-8)
    errors = rel(get(B.GET_L), L), rel(get(B.GET_R), R), rel(get(B.GET_PSH), P)
    print("    %d x %d %s: L %.1e R %.1e P %.1e" % (m, n, grad, *errors), flush=True)
    assert errors[0] <= 2 * 6e-8 and errors[1] <= 2 * 6e-8 and errors[2] <= 2e-6, errors


# bf16 gradients that the float32 matrix cores read, at an even and an odd address: four columns at a time, the last four again where three
# or fewer are left (131 and 255 columns), one by one where there are no four (2, 3); k short of a slab, and one more than a slab
@pytest.mark.parametrize("m,n", [(129, 131), (32, 255), (33, 130), (259, 3), (40, 2), (5, 64)])
@pytest.mark.parametrize("skew", [0, 1])
def test_bf16_gradients_on_the_float32_matrix_cores(m, n, skew):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m * n + skew)
    # epsilon of the size of the factor's eigenvalues: with 1e-6 the null space of R of one 32 x 255 gradient has 31 in the root where
    # the rest has 0.8, and what cancels there left 31 / 0.8 sqrt(255) 6e-8 = 4e-5 at worst (7e-6 measured)
    opt = B.Shampoo([(m, n)], 512, 0.99, 1.0, 0.25, 1, 0, grad_dtype=B.GRAD_BF16, precond_matrix_cores=B.MATRIX_CORES_FP32,
                    grafting_type=B.GRAFT_SGD)               # stage by stage at any size
    g = torch.empty(m * n + 8, device="cuda", dtype=torch.bfloat16)[skew:skew + m * n].view(m, n)
    g.copy_(torch.randn(m, n, device="cuda", generator=gen))
    opt.step([torch.zeros(m, n, device="cuda")], [g], 0.01, 0)
    get = lambda which: opt.get(0, 0, which).double()
    P = get(B.GET_LINV) @ g.double() @ get(B.GET_RINV)
    err = float((get(B.GET_PSH) - P).norm() / P.norm())
    print("    %d x %d: %.1e" % (m, n, err), flush=True)
    assert err <= 2e-6                                       # two sums of up to 259 values: 2 sqrt(259) 6e-8
