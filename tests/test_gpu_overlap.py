"""Small blocks on a stream of their own beside the stages of the others: the same bits as one after the other (which is how a
step runs while its stages are timed), eagerly and from a graph."""
import pytest

from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu

# 4.4e6 elements in blocks of 1024 and 76 x 1024, vectors and 40 small blocks
SHAPES = [(2124, 2048)] + [(96, 128)] * 40 + [(300,), (5000,)]


def run(graph, timed):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    opt = B.Shampoo(SHAPES, 1024, 0.99, 1e-12, 0.25, 100000, 0, momentum=0.9)
    w = [torch.zeros(s, device="cuda") for s in SHAPES]
    g = [torch.empty(s, device="cuda") for s in SHAPES]
    opt.set_timing(timed)

    def fill():
        for x in g:
            x.copy_(torch.randn(x.shape, device="cuda", generator=gen) * 1e-2)

    fill()
    opt.step(w, g, 0.01, 0)
    fill()
    opt.step(w, g, 0.01, 1000)
    out = []
    replay = None
    if graph:
        torch.cuda.synchronize()
        replay = torch.cuda.CUDAGraph()
        with torch.cuda.graph(replay):
            opt.step(w, g, 0.01, 1001)
    for k in range(3):                    # the program's own work and synchronisations between the replays
        fill()
        if graph:
            replay.replay()
        else:
            opt.step(w, g, 0.01, 1001 + k)
        torch.cuda.synchronize()
        out.append([x.clone() for x in w])
    return out


def test_same_bits():
    import torch
    want = run(False, True)
    for graph in (False, True):
        for step, (a, b) in enumerate(zip(want, run(graph, False))):
            assert all(torch.equal(x, y) for x, y in zip(a, b)), (graph, step)
