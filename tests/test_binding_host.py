"""The native binding and the interpreter lock, without a GPU: fake tensors pass its checks, and what it does next is seen.

Each case runs in a child process, which a lock that is not held ends with a nonzero status.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# fake tensors have no memory: on a machine with a GPU these calls would launch kernels on null pointers
pytestmark = pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="for machines without a GPU")

SETUP = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2512_07782_amd as g
with FakeTensorMode():
    alpha, c = (torch.empty(1, 1, 8, device="cuda") for _ in range(2))
"""


def child(code, *args):
    r = subprocess.run([sys.executable, "-c", code, *args], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, cwd=ROOT,
                       env=dict(os.environ, PYTHONPATH=ROOT), timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    return r.stdout


def test_an_error_inside_a_call_is_raised_with_the_lock_held():
    # outputs are given, so the first thing that fails is the look-up of the current stream, while other threads may run
    out = child(SETUP + """
for _ in range(3):
    try:
        g.gfwa_gate_prefix(alpha, c)
    except RuntimeError as e:
        print("raised:", e)
""")
    assert out.count("raised:") == 3, out


def test_outputs_are_allocated_without_the_lock(tmp_path):
    # an allocation may wait for the driver.  The allocation the binding calls is put in front of torch's, asks for the
    # lock's state and ends the process
    call_lib = os.path.join(ROOT, "paper_2512_07782_amd", "_gfwa_call.so")
    names = subprocess.run(["nm", "-D", "--undefined-only", call_lib], stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    (name,) = [n for n in names if "empty_cuda" in n]
    (tmp_path / "seen.c").write_text(f"""
        #include <stdio.h>
        #include <unistd.h>
        int PyGILState_Check(void);
        void allocation(void) __asm__("{name}");
        void allocation(void) {{ printf("lock held: %d\\n", PyGILState_Check()); fflush(stdout); _exit(0); }}
    """)
    lib = str(tmp_path / "seen.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", lib, str(tmp_path / "seen.c")], check=True)
    first = "import ctypes, sys\nctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)\n"
    assert "lock held: 0" in child(first + SETUP + "g.gfwa_gate_prefix(alpha)\n", lib)
