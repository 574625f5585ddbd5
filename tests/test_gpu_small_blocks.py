"""The step of a block of at most 128 x 128 in one workgroup, element by element against float64: sizes at the edges of its
tiles (32), of its two variants (64, 128), of its vectors (4), and both sides of the scale that it puts on a gradient."""
import numpy as np
import pytest

from paper_2309_06497_amd import binding as B
from paper_2309_06497_amd import workloads as wl
from test_gpu_parity import Pair

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 128), (2, 3), (5, 3), (3, 4), (33, 5), (64, 64), (63, 65), (65, 64), (32, 97), (97, 31), (128, 19), (37, 100), (96, 128), (128, 128)]


def f32(v):
    return float(np.float32(v))


def run(shape, bf16, beta1, sigma, steps=6):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    o = {"momentum": 0.9, "grad_dtype": B.GRAD_BF16 if bf16 else B.GRAD_F32}
    if beta1:
        o.update(beta1=beta1, use_bias_correction=True)
    # the roots are taken at the fourth step; the two after it are the ones that are looked at
    opt = B.Shampoo([shape], 128, 0.999, 1e-6 * sigma * sigma, 0.25, 1000, 3, **o)
    w = torch.randn(shape, device="cuda", generator=gen)
    grads = [(torch.randn(shape, device="cuda", generator=gen) * sigma).to(torch.bfloat16 if bf16 else torch.float32) for _ in range(steps)]
    for t, g in zip(range(997, 997 + steps), grads):
        opt.step([w], [g], 0.01, t)
    beta = f32(0.999)
    L = R = Gf = 0.0
    for g in grads:
        x = g.double()
        L = beta * L + (1.0 - beta) * (x @ x.T)
        R = beta * R + (1.0 - beta) * (x.T @ x)
        Gf = f32(beta1) * Gf + (1.0 - f32(beta1)) * x if beta1 else x
    if beta1:
        Gf = Gf / (1.0 - f32(beta1) ** (997 + steps))
    get = lambda which: opt.get(0, 0, which).double()
    P = get(B.GET_LINV) @ Gf @ get(B.GET_RINV)
    return opt, w, grads, (get(B.GET_L), L), (get(B.GET_R), R), (get(B.GET_PSH), P)


def off(pair):
    a, b = pair
    return float((a - b).norm() / b.norm())


# Factors: stored as float32 in each of the six steps, 2^-24 of an element each time (6 x 6e-8).
TOL_FACTOR = 3.6e-7
# Lbar G Rbar: two sums of at most 48 additions that are rounded to float32, 6e-8 each, at random: 6e-8 sqrt(96) = 5.8e-7;
# with a filter its six roundings of an element too.
TOL_P = 1e-6


@pytest.mark.parametrize("bf16,beta1", [(False, 0.0), (True, 0.0), (False, 0.9), (True, 0.9)])
@pytest.mark.parametrize("shape", SIZES)
def test_small_block_against_float64(shape, bf16, beta1):
    opt, _, _, L, R, P = run(shape, bf16, beta1, 1e-2)
    assert off(L) <= TOL_FACTOR and off(R) <= TOL_FACTOR and off(P) <= TOL_P, (off(L), off(R), off(P))
    assert (L[0] == L[0].T).all() and (R[0] == R[0].T).all()


@pytest.mark.parametrize("sigma", [1e-17, 1e-13, 1e13, 1e17])
def test_small_block_of_very_small_and_large_gradients(sigma):
    """Below 2^-40 and above 2^40 the block is scaled; the products still fit float32."""
    _, _, _, L, R, P = run((96, 40), False, 0.0, sigma)
    assert off(L) <= TOL_FACTOR and off(R) <= TOL_FACTOR and off(P) <= TOL_P, (off(L), off(R), off(P))


@pytest.mark.parametrize("bf16", [False, True])
def test_factors_are_whole_where_the_next_step_needs_them(bf16):
    """The step in one workgroup updates the lower triangles; a refresh, which goes stage by stage, reads more."""
    import torch
    shape = (104, 72)
    opt, w, grads, _, _, _ = run(shape, bf16, 0.0, 1e-2)
    opt.step([w], [grads[0]], 0.01, 2000)
    beta = f32(0.999)
    L = 0.0
    for g in grads + [grads[0]]:
        x = g.double()
        L = beta * L + (1.0 - beta) * (x @ x.T)
    got = opt.get(0, 0, B.GET_L).double()
    assert off((got, L)) <= 7 * 6e-8 and (got == got.T).all()
    lam, Q = np.linalg.eigh(got.cpu().numpy())
    root = (Q * (lam - min(lam[0], 0.0) + f32(1e-10)) ** -0.25) @ Q.T
    got = opt.get(0, 0, B.GET_LINV).double().cpu().numpy()
    assert np.linalg.norm(got - root) <= 1e-5 * np.linalg.norm(root)      # the bar of a root


@pytest.mark.parametrize("bf16", [False, True])
def test_filtered_parameter_of_small_and_larger_blocks(bf16):
    """200 x 200 in blocks of 150: the filter of the whole parameter is updated ahead of the stages of its larger blocks, and only read
    by the one workgroup of its 50 x 50 block, which updates that of the parameter beside it.  Bars of test_gpu_parity.py."""
    shapes = [(200, 200), (96, 64), (50,)]
    p = Pair(shapes, 150, 0.99, 3, eps=1e-6, bf16=bf16, beta1=0.9, bias_correction=True)
    for t in range(6):
        p.step(wl.gaussian_grads(shapes, 83, t, 1e-2), 0.01, t)
        p.check(t)


@pytest.mark.parametrize("count", [224, 225])
def test_as_many_parameters_as_a_launch_carries_pointers_of(count):
    """And one more, which takes them from the tables: the same bits as in two optimizers of half as many, whose buffers take turns too."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(31)
    shapes = [(24, 20), (7,), (5, 33)] * (count // 3) + [(40, 8)] * (count % 3)
    draw = lambda: [torch.randn(s, device="cuda", generator=gen) for s in shapes]
    w, g = [draw() for _ in range(2)], [draw() for _ in range(2)]
    v = [[x.clone() for x in ws] for ws in w]
    make = lambda s: B.Shampoo(s, 64, 0.99, 1e-6, 0.25, 100, 0, momentum=0.9)
    half = count // 2
    whole, parts = make(shapes), (make(shapes[:half]), make(shapes[half:]))
    for t in range(5):                    # the first one takes the roots; the others bring their pointers along or not
        whole.step(w[t % 2], g[t % 2], 0.01, t)
        parts[0].step(v[t % 2][:half], g[t % 2][:half], 0.01, t)
        parts[1].step(v[t % 2][half:], g[t % 2][half:], 0.01, t)
    assert all(torch.equal(x, y) for a, b in zip(w, v) for x, y in zip(a, b))
