"""Roots of buckets of many sizes in one refresh (csrc/group.h): every launch serves all of them, each at its own panel. Against
the fp64 oracle's roots of the same factors."""
import numpy as np
import pytest

from oracle import shampoo_oracle as so
from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu

MATRIX = [(B.GET_L, B.GET_LINV), (B.GET_R, B.GET_RINV)]
TENSOR = {3: MATRIX + [(B.GET_L2, B.GET_L2INV)], 4: MATRIX + [(B.GET_L2, B.GET_L2INV), (B.GET_L3, B.GET_L3INV)]}


# sizes on both sides of the kernels' classes: 32, 64 and 128 in LDS; panels of 256, 512 and 1024 rows
@pytest.mark.parametrize("shapes,block", [
    ([(20, 33), (64, 65), (128, 129), (130, 257), (300, 513)], 1024),
    ([(1056, 40), (161, 1025), (7, 128)], 2048),
    ([(700, 333)], 256),                                        # four buckets, the full one has two blocks
    ([(40, 130, 9), (16, 150, 3, 3), (200, 96)], 256),          # exponents 1/6 and 1/8 beside 1/4
])
def test_roots_of_a_refresh(shapes, block):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    opt = B.Shampoo(shapes, block, 0.99, 1e-12, 0.25, 1, 0)
    w = [torch.zeros(s, device="cuda") for s in shapes]
    for t in range(3):
        opt.step(w, [torch.randn(s, device="cuda", generator=gen) * 1e-2 for s in shapes], 0.01, t)
    table, buckets = opt.plan()
    assert buckets >= 3 and opt.status()["failed_roots"] == 0
    count = {}
    for row in table:
        p, flags = int(row[0]), int(row[7])
        k = count[p] = count.get(p, -1) + 1
        modes = flags >> 4 if flags & 4 else 2
        for factor, root in TENSOR[modes] if flags & 4 else MATRIX:
            a, x = opt.get(p, k, factor).cpu().numpy(), opt.get(p, k, root).cpu().numpy()
            want, _ = so.root_inverse(a, float(np.float32(1e-12)), 0.5 / modes)
            err = np.linalg.norm(x - want) / np.linalg.norm(want)
            print(f"    {shapes[p]} block {k} n={a.shape[0]}: {err:.1e}", flush=True)
            assert np.array_equal(x, x.T) and err <= 1e-5, (p, k, a.shape, err)      # as for one size at a time


def test_more_matrices_than_the_scratch_has_room_for():
    """190 matrices of 1024 and as many of 700 in one refresh, in two passes of equal size: some of the larger ones, then the rest of them
    and all of the smaller ones.  Against the roots of the same factors, one size at a time."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    m, n, count = 1024, 700, 190
    opt = B.Shampoo([(m, n)] * count, m, 0.99, 1e-12, 0.25, 1, 2)
    w = [torch.zeros(m, n, device="cuda") for _ in range(count)]
    for t in range(3):
        opt.step(w, [torch.randn(m, n, device="cuda", generator=gen) * 1e-2 for _ in range(count)], 0.01, t)
    assert opt.status() == {"refreshes": 1, "failed_roots": 0}
    for factor, root in MATRIX:
        a, x = (torch.stack([opt.get(p, 0, which) for p in range(count)]) for which in (factor, root))
        want = B.shampoo_root_inverse(a, 1e-12, 0.25)
        err = (x - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)
        print(f"    n={a.shape[1]}: {float(err.max()):.1e}", flush=True)
        assert float(err.max()) <= 2e-5      # both within the 1e-5 of test_roots_of_a_refresh
    opt.destroy()


@pytest.mark.parametrize("shapes", [[(1024, 704)] * 40, [(1024, 704)] * 150 + [(1024, 1024)] * 110], ids=["planes wait", "two sets of buckets"])
def test_directions_of_a_refresh(shapes):
    """Float32 gradients: the planes that the factor update has made either wait beside the scratch of the roots, or are made again in the
    memory that it has used."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(13)
    opt = B.Shampoo(shapes, 1024, 0.99, 1e-12, 0.25, 1, 2)
    w = [torch.zeros(s, device="cuda") for s in shapes]
    for t in range(4):
        g = [torch.randn(s, device="cuda", generator=gen) * 1e-2 for s in shapes]
        opt.step(w, g, 0.01, t)
    assert opt.status() == {"refreshes": 2, "failed_roots": 0}
    for p in (0, len(shapes) // 2, len(shapes) - 1):
        want = opt.get(p, 0, B.GET_LINV).double() @ g[p].double() @ opt.get(p, 0, B.GET_RINV).double()
        err = float((opt.get(p, 0, B.GET_PSH).double() - want).norm() / want.norm())
        print(f"    {shapes[p]}: {err:.1e}", flush=True)
        # two sums of 32 roundings to float32 each, 6e-8 sqrt(64) at random, by the norms of |Lbar| |G| |Rbar|, which is at most some ten times that of the product here
        assert err <= 5e-6, (p, err)
    opt.destroy()
