"""A kernel launch that fails is reported by the call that made it: every
launch of every entry point, on a HIP runtime that runs nothing."""

import pytest

import stub_common

BODY = '''
import numpy as np

def each_launch(call, ready=lambda: None):
    ready()
    assert fails(call) == 0, lib.estimator_last_error()
    ready()
    stub.stub_reset(-1)  # the launches of a call whose tables are there, unless ready() takes a new handle
    assert fails(call) == 0
    names = launched()
    for i, name in enumerate(names):
        ready()
        stub.stub_reset(i)
        status = fails(call)
        assert status == lib.EST_EDEVICE, (i, name, status)
        stub.stub_reset(-1)
    ready()
    assert fails(call) == 0  # nothing is left behind
    return len(names)
'''

# orders 1 and 2 with few particles on 256^3: the 32-bit general kernel and then the 64-bit walk;
# 16: one tile; 5 and 6: the general kernel alone
FORWARD = [(n, order, code, flags, 1) for n in (16, 32, 100, 256) for order in (1, 2, 4, 5)
           for code in (0, 1, 3) for flags in (0, 2)] + [
    (64, 6, 2, 0, 3), (64, 3, 1, 3, 2), (32, 4, 1, 1, 1)]


def test_forward_and_adjoint():
    out = stub_common.run(BODY + '''
total = 0
for n, order, code, flags, batch in %r:
    h = handle(n, order, code, batch, 5000, flags)
    if flags & lib.EST_FLAG_WEIGHTS:
        lib.estimator_set_weights(h, FAKE)
    off = FAKE if batch > 1 else None
    for dtype in (0, 1):
        total += each_launch(lambda: lib.estimator_deposit(h, FAKE, dtype, off, 5000))
        total += each_launch(lambda: lib.estimator_backward(h, FAKE, dtype, off, 5000, FAKE, 1, 8, FAKE))
    for choice in (0, 4, 43):  # the 64-bit format alone, both formats
        lib.estimator_set_launch(h, choice)
        total += each_launch(lambda: lib.estimator_deposit(h, FAKE, 0, off, 5000))
    deposit = lambda: lib.estimator_deposit(h, FAKE, 0, off, 5000)
    total += each_launch(lambda: lib.estimator_transform(h), deposit)
    deposit(), lib.estimator_transform(h)
    total += each_launch(lambda: lib.estimator_power(h, 1, 8, 0, FAKE, FAKE, FAKE))
    lib.estimator_destroy(h)
print(total)
''' % FORWARD)
    assert int(out) > 1000


def test_other_entry_points():
    """On a new handle each time: the tables of a first call are part of it."""
    stub_common.run(BODY + '''
def new():
    global h
    lib.estimator_destroy(h)
    h = handle(n, 4, code)

def forward():
    new()
    lib.estimator_deposit(h, FAKE, 0, None, 5000)
    lib.estimator_transform(h)

h = None
tri = np.array([(a, b, c) for a in range(1, 8) for b in range(1, a + 1) for c in range(max(1, a - b), b + 1)], np.int32)
for n, code in ((32, 0), (32, 1), (60, 1), (32, 2)):
    new()
    size = lib.estimator_bispectrum_workspace_bytes(h, 1, 4, len(tri))
    ws = np.zeros(size + 256, np.uint8)  # the job lists are copied to it
    at = (ws.ctypes.data + 255) // 256 * 256
    some = tri[tri[:, 0] <= 4]
    need = lib.estimator_direct_workspace_bytes(h, 100)
    each_launch(lambda: lib.estimator_power(h, 1, 8, 0, FAKE, FAKE, FAKE), forward)
    each_launch(lambda: lib.estimator_backward(h, FAKE, 0, None, 5000, FAKE, 1, 8, FAKE), new)
    each_launch(lambda: lib.estimator_export_delta(h, 0, FAKE), forward)
    each_launch(lambda: lib.estimator_sample_delta(h, 0, FAKE, 5, FAKE), forward)
    each_launch(lambda: lib.estimator_copy_grid(h, 1, 0, FAKE), lambda: (new(), lib.estimator_deposit(h, FAKE, 0, None, 5000)))
    each_launch(lambda: lib.estimator_spectrum_power(h, FAKE, None, 1, 8, 0.0, FAKE, FAKE, FAKE), new)
    each_launch(lambda: lib.estimator_graph_capture(h, FAKE, 0, None, 5000, 1, 8, 0, FAKE, FAKE, FAKE), new)
    each_launch(lambda: lib.estimator_direct_delta(h, FAKE, 0, 100, FAKE, need, FAKE), new)
    each_launch(lambda: lib.estimator_direct_delta_noalloc(h, FAKE, 1, 100, FAKE), new)
    each_launch(lambda: lib.estimator_autotune(h, FAKE, 0, None, 5000, 1, 8, 1), new)
    each_launch(lambda: lib.estimator_bispectrum(h, 0, 1, 4, some, len(some), at, size, FAKE, FAKE), forward)
''')


def test_creation():
    stub_common.run(BODY + 'each_launch(handle)\n')
