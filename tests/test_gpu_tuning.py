"""What the first context of a shape in a process costs: the trial launches that choose its tilings and its loop
traversal. In a process of its own, since a shape is tuned once."""
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

HEAD = """
import time, torch
from paper_1208_1186_amd import gf
def context(dims, precision):
    shape = tuple(reversed(dims)) + (4, 3, 3)
    u = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand(shape).contiguous()
    torch.cuda.synchronize()
    t = time.perf_counter()
    fx = gf.GaugeFixer(u, precision, check_every=10)
    return fx, 1e3 * (time.perf_counter() - t)
"""


def _child(code, repo_root):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, "-c", HEAD + code], capture_output=True, text=True, cwd=repo_root, timeout=100)
    print(r.stdout, r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    return r.stdout.split()


def test_first_large_context_costs_fewer_than_160_updates(repo_root):
    """At 32^4 in double a context with 12 launches a trial, alone or behind the launch that writes their input, costs
    160 to 230 updates; the alternatives differ by enough to tell with fewer (about 90 updates)."""
    cold, update = map(float, _child("""
context((4, 4, 4, 6), "fp64_18")  # library and device are set up
fx, cold = context((32, 32, 32, 32), "fp64_18")
fx.advance(20)
t = time.perf_counter()
fx.advance(100)
print(cold, 10 * (time.perf_counter() - t))
""", repo_root))
    assert cold < 160 * update
