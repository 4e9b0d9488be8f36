"""Host side of libfsest.so on a HIP runtime that runs nothing (hip_stub.c).

``run(body)`` executes ``body`` in a child process whose HIP calls go to the
stub, with these names defined: ``lib`` (the package), ``stub`` (the stub's
functions), ``handle(**config)``, ``launched()`` (names of the kernels
launched since the last ``stub.stub_reset``) and ``fails(call)`` (the status
of a call that raises, else 0).
"""

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PROLOGUE = '''
import ctypes, sys
sys.path.insert(0, %r)
import paper_1512_07295_amd as lib
stub = ctypes.CDLL(None)
stub.stub_kernel.restype = stub.stub_launched.restype = ctypes.c_char_p
FAKE = 1 << 30  # an aligned address that nothing reads

def handle(n_grid=32, order=4, interlace=1, batch=1, max_particles=5000, flags=0, workspace=FAKE):
    cfg = lib.make_config(n_grid, 500.0, order, interlace, batch, max_particles, flags)
    return lib.estimator_create(cfg, workspace, lib.estimator_workspace_bytes(cfg), 0)

def launched():
    return [stub.stub_launched(i).decode() for i in range(stub.stub_launches())]

def fails(call):
    try:
        call()
    except lib.FsestError as e:
        return e.status
    return 0
''' % ROOT


def run(body):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "hip_stub.so")
        subprocess.run(["gcc", "-O1", "-fPIC", "-shared", "-o", so, os.path.join(HERE, "hip_stub.c")], check=True)
        # no device for the parts of torch that see the real runtime
        preload = " ".join(filter(None, [so, os.environ.get("LD_PRELOAD")]))
        env = dict(os.environ, LD_PRELOAD=preload, HIP_VISIBLE_DEVICES="-1")
        out = subprocess.run([sys.executable, "-c", PROLOGUE + body], env=env, capture_output=True, text=True,
                             timeout=600)
    assert out.returncode == 0, out.stderr[-4000:]
    return out.stdout
