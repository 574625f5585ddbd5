"""Roots asked for without eigenvalues (csrc/root_tridiag.h, csrc/root_band.h) against the fp64 oracle, at the edges of
the kernels' size classes and on every kind of spectrum that is handled by a branch of its own."""
import numpy as np
import pytest

from oracle import shampoo_oracle as so
from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu

KINDS = ("single", "well", "low", "indefinite", "dead_rows", "diagonal", "zero")


def matrix(kind, n, rng):
    cols = {"single": n, "well": 4 * n, "low": max(1, n // 32)}.get(kind, n)
    g = rng.standard_normal((n, cols))
    a = g @ g.T * (1e-9 * n / cols)
    if kind == "low":
        a = g @ g.T + 1e-6 * np.eye(n)
    elif kind == "indefinite":
        a = (g + g.T) * 1e-3
    elif kind == "dead_rows":           # parameters that have never had a gradient
        a[::3] = 0.0
        a[:, ::3] = 0.0
    elif kind == "diagonal":
        a = np.diag(rng.standard_normal(n))
    elif kind == "zero":
        a = np.zeros((n, n))
    a = a.astype(np.float32)
    return (a + a.T) / np.float32(2)


def check(n, r, kinds=KINDS):
    import torch
    rng = np.random.default_rng(1000 + n)
    a = np.stack([matrix(k, n, rng) for k in kinds])
    x, failed = B.shampoo_root_inverse(torch.from_numpy(a).cuda(), 1e-12, r, False, True)
    x = x.cpu().numpy()
    assert not failed.cpu().numpy().any()
    for i, kind in enumerate(kinds):
        want, _ = so.root_inverse(a[i], float(np.float32(1e-12)), float(np.float32(r)))
        err = np.linalg.norm(x[i] - want) / np.linalg.norm(want)
        print(f"    n={n} r={r:.3f} {kind}: {err:.1e}", flush=True)
        assert np.array_equal(x[i], x[i].T)
        assert err <= 1e-5, (n, r, kind, err)


@pytest.mark.parametrize("n", [1, 2, 3, 17, 31, 32, 33, 63, 64, 65, 80, 127, 128])
def test_small_sizes(n):
    check(n, 0.25)


# no reflector, one, fewer than a tile of 16 holds, as many, one more
@pytest.mark.parametrize("n", [4, 5, 8, 14, 15, 16, 18, 19])
def test_sizes_around_one_tile(n):
    check(n, 0.25)


@pytest.mark.parametrize("n", [129, 160, 161, 255, 288, 544, 1056])
def test_band_sizes(n):
    check(n, 0.25)


@pytest.mark.parametrize("n,kinds", [(2048, ("low",)), (2017, ("single",))])
def test_largest_band_sizes(n, kinds):
    check(n, 0.25, kinds)


def test_exponents_of_the_band_path():
    for r in (1 / 6, 0.5):
        check(200, r)


@pytest.mark.parametrize("n", [33, 64, 100, 128, 129, 136, 144, 151, 160, 169, 200, 256, 291, 390, 512, 700])
def test_columns_that_depend_on_each_other(n):
    """All rows and columns alike but for a ridge (none for the smallest: epsilon serves as one): within a panel every
    reflection leaves 1e-16 of the next column, down to where squares are no longer numbers of full precision."""
    import torch
    scales = ((1.0, 1e-3), (0.37, 1e-3), (4.1e7, 1e-3), (2.5e-9, 0.0))
    a = np.stack([(c * (np.ones((n, n)) + ridge * np.eye(n))).astype(np.float32) for c, ridge in scales])
    x = B.shampoo_root_inverse(torch.from_numpy(a).cuda(), 1e-12, 0.25).cpu().numpy()
    for i in range(4):
        # J / n and I - J / n are the eigenprojections
        diag, off = a[i, 0, 0].astype(np.float64), a[i, 0, 1].astype(np.float64)
        eps, J = float(np.float32(1e-12)), np.full((n, n), 1.0 / n)
        want = (diag - off + eps) ** -0.25 * (np.eye(n) - J) + (diag + (n - 1) * off + eps) ** -0.25 * J
        err = np.linalg.norm(x[i] - want) / np.linalg.norm(want)
        print(f"    n={n} {scales[i]}: {err:.1e}", flush=True)
        assert err <= 1e-5, (scales[i], err)


@pytest.mark.parametrize("n", [40, 128, 129, 160, 512, 1000])
@pytest.mark.parametrize("lam", [(2e-10, 3e-10), (1e-10, 1.05e-10), (3e-11, 2e-10), (-2e-10, -1.9e-10), (-1e-10, 2e-11)])
def test_smallest_eigenvalues_close_to_each_other(n, lam):
    """A 2 x 2 block with two eigenvalues at 1e-10 of the largest, exact in float32, beside well-conditioned ones: the
    smaller one is handled by itself and has to be told from the other.  1e-5 of the root as everywhere here; float64
    resolves these eigenvalues (plus epsilon) to 1e-5 at worst."""
    import torch
    rng = np.random.default_rng(3000 + n)
    g = rng.standard_normal((n, 4 * n)) / np.sqrt(20.0 * n)
    a = (g @ g.T).astype(np.float32)
    i, j = n // 3, n - 2
    a[[i, j]] = 0.0
    a[:, [i, j]] = 0.0
    a[i, i] = a[j, j] = np.float32((lam[0] + lam[1]) / 2)
    a[i, j] = a[j, i] = np.float32((lam[1] - lam[0]) / 2)
    a = (a + a.T) / np.float32(2)
    x = B.shampoo_root_inverse(torch.from_numpy(a[None]).cuda(), 1e-12, 0.25)[0].cpu().numpy()
    # the oracle block by block: as a whole, float64 would move the small eigenvalues by as much as is tested here
    pair, rest = np.ix_([i, j], [i, j]), np.ix_(np.setdiff1d(np.arange(n), [i, j]), np.setdiff1d(np.arange(n), [i, j]))
    small = np.linalg.eigvalsh(a[pair].astype(np.float64))
    eps = float(np.float32(1e-12)) - min(small[0], 0.0)
    want = np.zeros((n, n))
    for blk in (pair, rest):
        l, q = np.linalg.eigh(a[blk].astype(np.float64))
        want[blk] = (q * (l + eps) ** -0.25) @ q.T
    err = np.linalg.norm(x - want) / np.linalg.norm(want)
    print(f"    n={n} {lam}: {err:.1e}", flush=True)
    assert err <= 1e-5, err


@pytest.mark.parametrize("n,r", [(160, 0.25), (160, 0.5), (224, 0.6), (256, 0.25), (256, 0.5), (480, 1 / 6), (512, 0.25), (544, 0.25), (1024, 0.25)])
def test_no_less_accurate_than_with_eigenvectors(n, r):
    """The same matrices with and without eigenvalues asked for, i.e. by block Jacobi and without eigenvectors: the error
    of the latter, in the mean over the batch, is no larger."""
    import torch
    rng = np.random.default_rng(2000 + n)
    for kind in ("single", "well", "low"):
        a = np.stack([matrix(kind, n, rng) for _ in range(4)])
        dev = torch.from_numpy(a).cuda()
        x, ref = B.shampoo_root_inverse(dev, 1e-12, r).cpu().numpy(), B.shampoo_root_inverse(dev, 1e-12, r, True)[0].cpu().numpy()
        want = np.stack([so.root_inverse(m, float(np.float32(1e-12)), float(np.float32(r)))[0] for m in a])
        err, bar = (np.mean([np.linalg.norm(y[i] - want[i]) / np.linalg.norm(want[i]) for i in range(4)]) for y in (x, ref))
        print(f"    n={n} r={r:.3f} {kind}: {err:.2e}, with eigenvectors {bar:.2e}", flush=True)
        assert err <= bar * 1.05, (kind, err, bar)     # 5 %: the spread of the mean of four


@pytest.mark.parametrize("r", [1 / 6, 1 / 3, 0.5])
def test_exponents(r):
    check(72, r)


@pytest.mark.parametrize("n", [48, 160])
def test_non_finite_matrices_keep_their_output(n):
    import ctypes
    import torch
    a = np.stack([matrix("well", n, np.random.default_rng(5))] * 3)
    a[1, 7, 9] = a[1, 9, 7] = np.nan
    dev = torch.from_numpy(a).cuda()
    x = torch.full_like(dev, 7.0)
    failed = torch.zeros(3, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.lib().shampoo_root_inverse_workspace_bytes(n, 3), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = B.lib().shampoo_root_inverse(p(dev), n, 3, 1e-12, 0.25, p(x), None, p(failed), p(ws), ws.numel(),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0 and failed.tolist() == [0, 1, 0]
    assert bool((x[1] == 7.0).all()) and bool((x[0] != 7.0).all())
