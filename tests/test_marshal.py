"""csrc/marshal.cpp without a GPU: what the tensor library throws comes back as a Python exception and does not end the
process.  In processes of their own, so that one that does end is seen as a failure."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = "import torch\nfrom paper_2309_06497_amd import _marshal\nassert not torch.cuda.is_available()\n"


def run(code):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", CUDA_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    return subprocess.run([sys.executable, "-c", HEAD + code], env=env, capture_output=True, text=True, timeout=300)


@pytest.mark.parametrize("what,shapes,tensors", [
    ("no device to ask for its stream", "[]", "[]"),
    ("a tensor without storage", "[(2, 3)]", "fake()"),
])
def test_an_exception_stays_an_exception(what, shapes, tensors):
    p = run(f"""
from torch._subclasses.fake_tensor import FakeTensor, FakeTensorMode
def fake():
    with FakeTensorMode() as mode:
        return [FakeTensor(mode, torch.empty(2, 3, device="meta"), torch.device("cuda", 0))]
s = _marshal.make(0, 0, 0, False, {shapes})
ts = {tensors}
try:
    _marshal.step(s, ts, ts, 0.1, 0)
except Exception as e:
    print("raised", type(e).__name__, e)
""")
    assert p.returncode == 0 and p.stdout.startswith("raised "), (what, p.returncode, p.stdout, p.stderr[-500:])


def test_argument_errors_name_the_parameter():
    p = run("""
s = _marshal.make(0, 0, 0, False, [(2, 3)])
t = torch.zeros(2, 3)
for ps, gs in (([t], []), ([t], [t]), ([1], [t]), (1, [t])):
    try:
        _marshal.step(s, ps, gs, 0.1, 0)
    except (ValueError, TypeError) as e:
        print(type(e).__name__, e)
""")
    assert p.returncode == 0, p.stderr[-500:]
    assert p.stdout.splitlines() == ["ValueError one parameter and one gradient tensor per declared parameter",
                                     "ValueError parameter 0: tensors must live on the optimizer's device",
                                     "ValueError parameter 0: parameters and gradients are tensors",
                                     "TypeError params is a sequence of tensors"]
