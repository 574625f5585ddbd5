"""Tensor blocks whose Gram matrices are formed in ranges, and float32 gradients split into planes, against the
oracle (bars of test_gpu_parity.py) and, element by element, against float64."""
import numpy as np
import pytest

from paper_2309_06497_amd import binding as B
from paper_2309_06497_amd import workloads as wl
from test_gpu_parity import Pair, TensorPair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last,bf16", [(2, False), (9, True), (15, False), (16, False), (17, False)])
def test_last_dimension_around_the_narrow_gram_kernel(last, bf16):
    """Row counts that 16 does not divide, columns up to and just above one 16-wide tile; the first and
    the middle unfolding (k = 24 * last ...) are cut into one range, several, and a short last one."""
    shapes = [(20, 24, last), (7, 23, last), (9,)]
    p = TensorPair(shapes, 24, 0.99, 2, bf16=bf16)
    for t in range(3):
        p.step(wl.gaussian_grads(shapes, 71, t, 1e-2), 0.01, t)
        p.check(t)


@pytest.mark.parametrize("shape,b", [((72, 64, 3, 3), 128), ((128, 100, 3, 3), 128), ((128, 96, 5, 5), 128), ((144, 64, 3, 3), 256)])
def test_long_unfoldings_that_the_ranges_do_not_divide(shape, b):
    """One block that is the largest of its set, so that the scratch is no larger than its own m n; the number of
    ranges is bounded by that scratch, and k is no multiple of it."""
    shapes = [shape]
    p = TensorPair(shapes, b, 0.99, 2)
    for t in range(2):
        p.step(wl.gaussian_grads(shapes, 75, t, 1e-2), 0.01, t)
        p.check(t)


@pytest.mark.parametrize("dim,which", [(0, B.GET_L), (1, B.GET_L2)])
def test_sums_of_the_ranges_are_kept_in_float64(dim, which):
    """One inner product over 9 ranges of 128 values of k: 2^25 + 1 in the first one, -2^25 in the last.  Every 16 products
    add up exactly in float32; 2^25 + 1 does not fit one."""
    import torch
    opt = B.Shampoo([(128, 128, 9)], 128, 1.0, 1e-12, 0.25, 1000, 1)
    u = np.zeros((128, 1152), np.float32)
    u[0] = 1.0
    u[1, :16], u[1, 32], u[1, -16:] = 2.0 ** 21, 1.0, -2.0 ** 21
    g = np.ascontiguousarray(np.moveaxis(u.reshape(128, 128, 9), 0, dim))
    opt.step([torch.zeros(128, 128, 9, device="cuda")], [torch.from_numpy(g).cuda()], 0.0, 0)
    F = opt.get(0, 0, which).cpu().numpy()
    assert F[0, 0] == 1152.0 and F[0, 1] == 1.0 and F[1, 0] == 1.0


def test_tensors_of_different_order_whose_blocks_measure_the_same():
    shapes = [(6, 8, 9), (6, 8, 9, 9), (6, 17, 9)]
    p = TensorPair(shapes, 8, 0.99, 1)
    for t in range(2):
        p.step(wl.gaussian_grads(shapes, 77, t, 1e-1), 0.01, t)
        p.check(t)


def test_more_tensors_than_one_copy_launch_holds():
    shapes = [(3, 5, 7), (4, 6, 2), (5, 5, 5)] * 9 + [(6, 7)]
    p = TensorPair(shapes, 6, 0.99, 1)
    for t in range(2):
        p.step(wl.gaussian_grads(shapes, 72, t, 1e-2), 0.01, t)
        p.check(t)


@pytest.mark.parametrize("shape,decades", [((256, 384), (8, 0)), ((392, 144), (0, 12)), ((152, 264), (10, 10))])
def test_small_rows_and_columns_keep_their_accuracy(shape, decades):
    """Rows (columns) that are many decades below the largest.  Every element of a factor, measured by the norms of the
    two rows it is a product of: 2^-24 for the float32 it is stored in; the matrix cores add up 32 values of
    k in 12 steps, 12 x 2^-24 of their share at worst; 2^-24 for the products left out: 14 x 2^-24, once per gradient.
    Every element of Lbar G Rbar, measured by |Lbar| |G| |Rbar|: a rounding per 16 values of k in both products, and
    in each 2^-24 for the products left out, for the last sum and for the result."""
    import torch
    m, n = shape
    beta = float(np.float32(0.999))
    opt = B.Shampoo([shape], 512, 0.999, 1e-12, 0.25, 1000, 0)
    w = [torch.zeros(shape, device="cuda")]
    L, R = np.zeros((m, m)), np.zeros((n, n))
    steps = 2
    for t in range(steps):
        g = np.random.default_rng(80 + t).standard_normal(shape) * 1e-3
        g *= 10.0 ** (-decades[0] * np.arange(m) / m)[:, None] * 10.0 ** (-decades[1] * np.arange(n) / n)[None, :]
        g = g.astype(np.float32)
        opt.step(w, [torch.from_numpy(g).cuda()], 0.0, t)
        g = g.astype(np.float64)
        L = beta * L + (1.0 - beta) * g @ g.T
        R = beta * R + (1.0 - beta) * g.T @ g
    for which, want in ((B.GET_L, L), (B.GET_R, R)):
        got = opt.get(0, 0, which).cpu().numpy()
        d = np.sqrt(np.diag(want))
        err = np.abs(got - want) / np.outer(d, d)
        assert np.array_equal(got, got.T)
        assert err.max() <= 14 * steps * 2.0 ** -24, (which, err.max(), np.unravel_index(err.argmax(), err.shape))
    Li, Ri = (opt.get(0, 0, which).cpu().numpy().astype(np.float64) for which in (B.GET_LINV, B.GET_RINV))
    P = opt.get(0, 0, B.GET_PSH).cpu().numpy()
    err = np.abs(P - Li @ g @ Ri) / (np.abs(Li) @ np.abs(g) @ np.abs(Ri))
    steps_of = lambda k: 2 * -(-k // 32)
    assert err.max() <= (steps_of(m) + steps_of(n) + 6) * 2.0 ** -24, (err.max(), np.unravel_index(err.argmax(), err.shape))


@pytest.mark.parametrize("bf16", [False, True])
def test_factors_of_very_small_gradients(bf16):
    """Gradients of 3e-20: their scale is 2^76, its square is beyond float32, the factors (2e-37 a gradient) are not."""
    shapes = [(256, 384)]
    p = Pair(shapes, 512, 1.0, 1000, eps=1e-30, eps_g=1e-30, bf16=bf16)
    for t in range(3):
        p.step(wl.gaussian_grads(shapes, 76, t, 3e-20), 0.01, t)
    for which, want in ((B.GET_L, p.ora.L), (B.GET_R, p.ora.R)):
        got = p.gpu.get(0, 0, which).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - want[0][0]) <= 1e-5 * np.linalg.norm(want[0][0])


def test_more_blocks_than_the_planes_have_room_for():
    """181 blocks of 1024 x 1024, whose planes are made for 91 and then for 90 at a time: the blocks at the edges of the two
    parts, against float64 products of the same values."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    n, count = 1024, 181
    opt = B.Shampoo([(n, n * count)], n, 0.999, 1e-12, 0.25, 1000, 0)
    g = torch.randn(n, n * count, generator=gen, device="cuda") * torch.logspace(-4, -2, n * count, device="cuda")
    opt.step([torch.zeros_like(g)], [g], 0.0, 0)
    rel = lambda a, b: float((a.double() - b).norm() / b.norm())
    alpha = 1.0 - float(np.float32(0.999))
    for k in (0, 90, 91, 180):
        blk = g[:, n * k:n * (k + 1)].double()
        assert rel(opt.get(0, k, B.GET_L), alpha * blk @ blk.T) <= 1e-6, k
        assert rel(opt.get(0, k, B.GET_R), alpha * blk.T @ blk) <= 1e-6, k
        want = opt.get(0, k, B.GET_LINV).double() @ blk @ opt.get(0, k, B.GET_RINV).double()
        assert rel(opt.get(0, k, B.GET_PSH), want) <= 2e-5, k
    opt.destroy()


@pytest.mark.parametrize("name,sigma,eps,span", [("tiny", 1e-15, 1e-30, False), ("huge", 1e10, 1e20, False), ("rows", 1e-3, 1e-9, True)])
def test_float32_gradients_in_planes(name, sigma, eps, span):
    """Blocks with ragged tiles and ragged k (136 = 128 + 8, 264 = 256 + 8, k % 32 of 8, 16 and 24) whose gradients
    are tiny, huge, or span six decades from row to row, and a zero block: factors, products, directions, by the norms of
    whole blocks (test_small_rows_and_columns_keep_their_accuracy looks at the small rows by themselves)."""
    shapes = [(256, 384), (392, 144), (152, 264)]
    p = Pair(shapes, 256, 0.999, 1, eps=eps, eps_g=sigma * 1e-7)
    for t in range(3):
        g = wl.gaussian_grads(shapes, 73, t, sigma)
        if span:
            for x in g:
                x *= (10.0 ** (-6.0 * np.arange(x.shape[0]) / x.shape[0]))[:, None].astype(np.float32)
            g[0][:, 256:] = 0.0
        p.step(g, 0.01, t)
        worst, _ = p.check(t)
        assert worst["gemm"] <= 2e-5, worst
    for w in p.w_gpu:
        assert np.isfinite(w.cpu().numpy()).all()


def test_filtered_gradients_in_planes():
    shapes = [(256, 384), (392, 144), (152, 264)]
    for bf16 in (False, True):
        p = Pair(shapes, 256, 0.999, 1, bf16=bf16, beta1=0.9, weight_decay=0.05, bias_correction=True, grafting="adam")
        for t in range(3):
            p.step(wl.gaussian_grads(shapes, 74, t, 1e-2), 0.01, t)
            p.check(t)


def test_buckets_whose_scratch_does_not_fit_side_by_side():
    """Four buckets of 90 blocks, 1.1 GB of planes each: two sets of two that use the same scratch one after the other."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    shapes = [(m, 1024 * 90) for m in (1024, 1016, 1008, 1000)]
    opt = B.Shampoo(shapes, 1024, 0.999, 1e-12, 0.25, 1000, 3, momentum=0.9)
    w = [torch.zeros(s, device="cuda") for s in shapes]
    beta = float(np.float32(0.999))
    L = [0.0] * 4
    for t in (998, 999, 1000, 1001):           # roots at the third, the fourth is looked at
        g = [torch.randn(s, device="cuda", generator=gen) * 1e-2 for s in shapes]
        for i in range(4):
            x = g[i][:, 89 * 1024:].double()
            L[i] = beta * L[i] + (1.0 - beta) * (x @ x.T)
        opt.step(w, g, 0.01, t)
    for i in range(4):
        get = lambda which: opt.get(i, 89, which).double()
        P = get(B.GET_LINV) @ g[i][:, 89 * 1024:].double() @ get(B.GET_RINV)
        factor, direction = float((get(B.GET_L) - L[i]).norm() / L[i].norm()), float((get(B.GET_PSH) - P).norm() / P.norm())
        # float32 storage in each of four steps; the error that gemm_f16x2.h states for such products is 2.8e-7
        assert factor <= 4 * 6e-8 and direction <= 1e-6, (i, factor, direction)
