"""Which tensors a step works on where some steps are recorded into graphs: an eager one on those it is given, a replay on those it was
recorded with.  Against the same steps without a graph."""
import pytest

from paper_2309_06497_amd import binding as B

pytestmark = pytest.mark.gpu


class Run:
    def __init__(self, shapes, block):
        import torch
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(23)
        self.opt = B.Shampoo(shapes, block, 0.99, 1e-6, 0.25, 100, 0, momentum=0.9)
        draw = lambda: [torch.randn(s, device="cuda", generator=self.gen) * 1e-2 for s in shapes]
        self.w, self.g = [draw() for _ in range(2)], [draw() for _ in range(2)]      # two sets of buffers
        self.replay = None

    def eager(self, t, which):
        import torch
        self.opt.step(self.w[which], self.g[which], 0.01, t)
        torch.cuda.synchronize()

    def record(self, t, which):
        import torch
        self.replay = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.replay):
            self.opt.step(self.w[which], self.g[which], 0.01, t)

    def replayed(self):
        import torch
        self.replay.replay()
        torch.cuda.synchronize()


def same(a, b):
    import torch
    return all(torch.equal(x, y) for v, u in zip(a.w, b.w) for x, y in zip(v, u))


def test_refresh_after_a_recorded_one_that_was_not_replayed():
    """Ordinary steps of small blocks bring their pointers along; the first reader of the tables is recorded, the second is not."""
    shapes = [(96, 128), (40,), (30, 70)]
    want, got = Run(shapes, 128), Run(shapes, 128)
    for r in (want, got):
        r.eager(100, 0)
        r.eager(101, 1)
    got.record(200, 1)
    for r in (want, got):
        r.eager(300, 1)
        r.eager(301, 0)
    assert same(want, got)


@pytest.mark.parametrize("shapes,block", [([(300, 128), (50,)], 256), ([(40, 24, 9), (20, 30)], 32)])
def test_replays_between_eager_steps_on_other_tensors(shapes, block):
    """No refresh and no bias correction: what a step does depends on its tensors alone, so that a replay is the step it repeats."""
    want, got = Run(shapes, block), Run(shapes, block)
    for r in (want, got):
        r.eager(0, 0)
        r.eager(1, 0)
    got.record(2, 0)
    t = 3
    for _ in range(3):
        want.eager(t, 0)
        got.replayed()
        for k in (1, 2):
            for r in (want, got):
                r.eager(t + k, 1)
        t += 3
    assert same(want, got)
