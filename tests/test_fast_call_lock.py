"""The interpreter's lock in the binding's native calls, on the CPU: tensors that say they are on a GPU and an entry point that
notes who holds the lock (tests/fast_call_host.cpp).  In a process of its own: Python objects touched without the lock end it."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = """
import importlib.util, sys
import torch
sys.path.insert(0, sys.argv[1])
from paper_1802_04730_amd import tc355
tc355.lib()
fast = tc355._FAST
spec = importlib.util.spec_from_file_location("fast_call_host", sys.argv[2])
host = importlib.util.module_from_spec(spec)
spec.loader.exec_module(host)
f = lambda *s: host.tensor("f", *s)
ws = host.tensor("b", 64)
calls = [
    (fast.tbmm, [f(3, 5, 9), f(3, 7, 9), f(3, 5, 7)]),
    (fast.tbmm_ws, [f(3, 5, 9), f(3, 7, 9), f(3, 5, 7), ws]),
    (fast.mlp, [f(3, 6), [f(5, 6), f(4, 5)], (f(5), f(4)), [None, f(3, 4)], ws]),
    (fast.gconv, [f(2, 3, 4, 8, 9), f(3, 5, 4, 3, 2), f(15), f(2, 3, 5, 6, 8)]),
    (fast.gconv, [f(2, 3, 4, 8, 9), f(3, 5, 4, 3, 2), None, f(2, 3, 5, 6, 8)]),
    (fast.kron, [f(3, 4), f(5, 6), f(2, 4, 6), f(2, 3, 5)]),
    (fast.sconv, [f(2, 3, 9, 8), f(4, 3, 3, 3), f(4), f(2, 4, 4, 6), 2, 1]),
    (fast.lut, [[f(9, 6), f(9, 6)], [host.tensor("i", 4, 2), host.tensor("i", 4, 3)], [f(4, 6), f(4, 6)]]),
]
for n, (call, args) in enumerate(calls):
    assert call(host.entry(), *args, 1) == 0 and host.count() == (n + 1, 0), (call, host.count())
    for no_entry in (None, "x", 1.5, object(), 1 << 80, -(1 << 80)):
        assert call(no_entry, *args, 1) == -1, (call, no_entry)
    if isinstance(args[0], torch.Tensor):
        assert call(host.entry(), torch.zeros(args[0].shape), *args[1:], 1) == -1  # one argument on the CPU
    assert host.count() == (n + 1, 0)
print("as expected")
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from paper_1802_04730_amd import build

    out = str(tmp_path_factory.mktemp("fast") / "fast_call_host.so")
    subprocess.run(build.torch_module_command(os.path.join(ROOT, "tests", "fast_call_host.cpp")) + ["-o", out], check=True)
    return out


def test_calls_are_made_without_the_lock_and_nothing_else_is(host):
    r = subprocess.run([sys.executable, "-c", CALLS, ROOT, host], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "as expected" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])
