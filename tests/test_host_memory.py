"""Host memory that runs out inside an entry point is an error code, not an exception through the C boundary.  In a process of its
own, so that one that ends is seen as a failure."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# 2^24 blocks of 1 x 1, of which a plan needs a gigabyte, under a limit of 128 MB more than the process has
CODE = """
import resource
from paper_2309_06497_amd import binding as B
cfg = B.make_config([(4096, 4096)], 1, 0.999, 1e-12, 0.25, 100)
small = B.make_config([(64, 64)], 32, 0.999, 1e-12, 0.25, 100)
B.lib()
pages = int(open("/proc/self/statm").read().split()[0])
limit = pages * resource.getpagesize() + (128 << 20)
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
try:
    B.shampoo_plan(cfg)
except B.ShampooError as e:
    print("code", e.code)
print(B.shampoo_workspace_bytes(cfg), len(B.shampoo_plan(small)[0]))
"""


def test_out_of_host_memory_is_an_error_code():
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", CUDA_VISIBLE_DEVICES="", PYTHONPATH=ROOT)
    p = subprocess.run([sys.executable, "-c", CODE], env=env, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.split("\n")[:2] == ["code -6", "0 4"], (p.returncode, p.stdout, p.stderr[-500:])
