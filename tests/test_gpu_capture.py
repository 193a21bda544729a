"""A call captured into a graph after one eager call at the same length with the
other sample type: every table the captured call needs is on the device by then.
In a process of its own, whose tables are those of that one call."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = r"""
import torch
import paper_1509_00186_amd as cdd
first, second, N = %r, %r, %d
nchan, f, bw, dm = 4, 330.0, 0.08, 3.0
def record(kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randint(-60, 61, (3 * N, nchan, 2), generator=g, device="cuda", dtype=torch.int8)
    return v if kind == "int8" else torch.view_as_complex(v.float())
cdd.dedisperse_noalloc(record(first, 1), f, bw, dm, N, 4)
v = record(second, 2)
out = {k: t for k, t in cdd.dedisperse_noalloc(record(first, 1), f, bw, dm, N, 4).items()
       if k in ("I", "cov")}
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    cdd.dedisperse_noalloc(v, f, bw, dm, N, 4, out=out)
for seed in (2, 3, 4):
    v.copy_(record(second, seed))
    want = cdd.dedisperse(v, f, bw, dm, N, 4)
    torch.cuda.synchronize()
    out["I"].zero_()
    out["cov"].zero_()
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(out["I"], want["I"]) and torch.equal(out["cov"], want["cov"]), seed
print("captured and replayed")
"""


@pytest.mark.parametrize("first,second", [("complex64", "int8"), ("int8", "complex64")])
def test_capture_after_a_call_of_the_other_type(first, second):
    print("case: capture of", second, "after", first, flush=True)
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", SCRIPT % (first, second, 8192)], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "captured and replayed" in r.stdout
