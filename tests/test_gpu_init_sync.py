"""init makes one host round trip, whatever form the couplings take: its calls
of hipStreamSynchronize are counted by a library of the test's own that stands
before the HIP runtime in a fresh process's symbol order."""
import os
import subprocess
import sys

import pytest

from gpu_common import announce, ensure_built

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = r"""
typedef int (*sync_fn)(void *);
static sync_fn target;
static int calls;
void count_target(void *f) { target = (sync_fn)f; calls = 0; }
int count_calls(void) { return calls; }
int hipStreamSynchronize(void *stream) { ++calls; return target(stream); }
"""

PROGRAM = r"""
import ctypes, sys
counter = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import torch
from paper_2305_07187_amd import instances, spring_ising as si
si.load_library()
hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
counter.count_target.argtypes = [ctypes.c_void_p]
counter.count_target(ctypes.cast(ctypes.CDLL(hip).hipStreamSynchronize, ctypes.c_void_p))
for n, r, kind in ((100, 8, "pm1"), (700, 1001, "pm1"), (700, 100, "gauss"), (700, 961, "gauss")):
    J = torch.from_numpy(instances.make_J(n, kind, 1)).float().cuda()
    x = torch.from_numpy(instances.make_x0(n, r, 1)).cuda()
    torch.cuda.synchronize()
    before = counter.count_calls()
    ctx = si.spring_ising_init(n, r, J, x, None, si.spring_ising_default_params(10))
    calls = counter.count_calls() - before
    torch.cuda.synchronize()
    si.spring_ising_destroy(ctx)
    print("calls", n, r, kind, calls, flush=True)
"""


def test_init_synchronises_once(tmp_path):
    ensure_built()
    announce("host round trips of init")
    src, lib, prog = tmp_path / "count.c", tmp_path / "count.so", tmp_path / "program.py"
    src.write_text(COUNTER)
    prog.write_text(PROGRAM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = subprocess.run([sys.executable, str(prog), str(lib), ROOT], capture_output=True, text=True, timeout=180)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]
    lines = [l.split() for l in r.stdout.splitlines() if l.startswith("calls")]
    assert len(lines) == 4 and all(l[-1] == "1" for l in lines), lines
