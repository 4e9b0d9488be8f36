"""Which kernels a call takes follows from the call itself (CPU, on the stub)."""

import pytest

import stub_common

pytest.importorskip("paper_1512_07295_amd", reason="libfsest.so not built")

SHAPES = '''
def shapes(n_grid, order, code, batch, room, n, weights=False):
    h = handle(n_grid, order, code, batch, room, lib.EST_FLAG_WEIGHTS if weights else 0)
    if weights:
        lib.estimator_set_weights(h, FAKE)
    stub.stub_reset(-1)
    lib.estimator_deposit(h, FAKE, 0, FAKE if batch > 1 else None, n)
    out = [(name, stub.stub_grid(i, 0), stub.stub_block(i)) for i, name in enumerate(launched())]
    lib.estimator_destroy(h)
    return out
'''


def test_room_of_the_handle_does_not_matter():
    """A handle with room for many particles launches for few what one with
    room for just these does."""
    stub_common.run(SHAPES + '''
for n_grid, batch in ((16, 1), (20, 1), (64, 1), (64, 5), (128, 1), (256, 1), (480, 1), (1024, 1)):
    for order in range(1, 7):
        if n_grid == 20 and order == 6:
            continue
        for code in (0, 1, 3):
            for n in (1, 5000, 100003, 1 << 22):
                own = shapes(n_grid, order, code, batch, n, n)
                for room in (n + 1, 16 * n, 1 << 27):
                    assert shapes(n_grid, order, code, batch, room, n) == own, (n_grid, batch, order, code, n, room)
''')


def test_fewer_particles_never_take_more_super_buckets():
    """The room's workspace holds the histograms of every smaller call: the
    super-buckets (a workgroup each in the bucket pass, 64 per workgroup of the
    column scan) grow with the particles."""
    stub_common.run(SHAPES + '''
def supers(shape):
    scan = [g for name, g, _ in shape if "k_sup_colscan" in name]
    fine = [g for name, g, _ in shape if "k_sort_fine" in name]
    return scan[0] if scan else 0, fine[0] if fine else 0

for n_grid, batch in ((20, 1), (64, 3), (100, 1), (256, 1), (300, 2), (320, 1), (512, 1), (1024, 1)):
    for order in (1, 2, 4, 5):
        for code in (0, 1):
            for weights in (False, True):
                last = (0, 0)
                for n in sorted({1, 500, 3000, 60000, 70000, 1 << 20, 1 << 22, 1 << 23, 1 << 24, 1 << 25, 1 << 27, 1 << 30}
                                | {n_grid ** 3 * batch // k for k in (64, 33, 31, 17, 15, 13, 11, 9, 7, 5, 4, 3, 1)}):
                    now = supers(shapes(n_grid, order, code, batch, n, n, weights))
                    assert now[0] >= last[0] and now[1] >= last[1], (n_grid, batch, order, code, weights, n)
                    last = now
''')


def test_sparse_grids_take_the_general_deposit():
    """(n_grid, batch, order, interlace, masses, cells per particle, general):
    both sides of each line, and both kinds of kernel in the 64-bit format."""
    stub_common.run(SHAPES + '''
lines = []
for n_grid, batch in ((512, 1), (400, 1), (128, 16), (64, 128)):
    for code, per in ((0, (4, 12, 12, 16)), (1, (4, 8, 16, 32 if n_grid >= 400 else None)), (2, (8, 12, 16, 32)), (3, (8, 12, 16, 32))):
        for order in (1, 2, 3, 4):
            lines.append((n_grid, batch, order, code, False, per[order - 1]))
    lines += [(n_grid, batch, 4, 0, True, 32), (n_grid, batch, 3, 0, True, 12), (n_grid, batch, 4, 1, True, 32)]
for order in (1, 2, 3, 4):
    lines += [(256, 1, order, 1, True, 32), (256, 1, order, 1, False, 64 if order == 3 else None), (256, 1, order, 3, False, 32),
              (160, 1, order, 0, False, 16), (200, 1, order, 2, False, 64), (96, 5, order, 0, False, 16)]
    lines += [(128, 1, order, code, False, None) for code in range(4)] + [(240, 1, order, 1, False, None)]
for n_grid, batch, order, code, masses, per in lines:
    cells = batch * n_grid ** 3
    counts = [(cells // per, True), (cells // per + 1, False)] if per else [(cells // 1000, False), (cells // 64, False), (cells, False)]
    if per and code and order >= 3:  # next to empty
        edge = -(-cells // (1024 if code == 1 else 2048))
        counts += [(edge, True), (edge - 1, False)]
    for n, general in counts:
        names = [name for name, _, _ in shapes(n_grid, order, code, batch, n, n, masses) if "k_deposit" in name]
        first = "k_depositILi%dELi%dELb0" % (order, min(code, 2)) if general else "k_deposit_walkILi%dELi%dELb0" % (order, min(code, 2))
        assert all(first in a and "k_deposit_walkILi%d" % order in b and "ELb1ELb" in b for a, b in zip(names[::2], names[1::2])), \\
            (n_grid, batch, order, code, masses, n, names)
''')


def test_every_deposit_kernel_is_reached():
    """No kernel of the deposit is compiled that no call can launch."""
    out = stub_common.run(SHAPES + '''
stub.stub_kernel.restype = ctypes.c_char_p
seen = set()
for n_grid, batch, n in ((16, 1, 100), (64, 1, 100), (40, 1, 100), (512, 1, 10 ** 6), (500, 1, 10 ** 6)):
    for order in range(1, 7):
        for code in (0, 1, 2):
            for weights in (False, True):
                seen |= {name for name, _, _ in shapes(n_grid, order, code, batch, n, n, weights)}
names = {stub.stub_kernel(i).decode() for i in range(stub.stub_kernels())}
print(sorted(name for name in names - seen if "k_deposit" in name))
''')
    assert out.strip() == "[]"


def test_masses_take_larger_super_buckets():
    """(particles, super-buckets without and with masses): 4K and 16K particles
    each, 64 super-buckets per workgroup of the column scan."""
    stub_common.run(SHAPES + '''
for n_grid, n, plain, masses in ((256, 1 << 24, 4096, 512), (512, 1 << 24, 4096, 512), (480, 360 ** 3, 8000, 1728), (256, 1 << 20, 512, 512),
                                  (300, 300 ** 3, 3375, 3375), (300, 15 << 20, 3375, 125)):
    for weights, count in ((False, plain), (True, masses)):
        scan = [g for name, g, _ in shapes(n_grid, 4, 1, 1, n, n, weights) if "k_sup_colscan" in name]
        assert scan == [-(-count // 64)], (n_grid, n, weights, scan)
''')


def test_few_particles_keep_workgroups_in_the_bucket_pass():
    """Its workgroups write the offsets of every bucket, at most 512 each here."""
    stub_common.run(SHAPES + '''
for n_grid, batch, least in ((64, 1, 8), (128, 1, 64), (256, 1, 64), (64, 8, 64), (512, 1, 512)):
    for n in (1, 100, 4096):
        fine = [g for name, g, _ in shapes(n_grid, 4, 1, batch, 1 << 22, n) if "k_sort_fine" in name]
        assert fine[0] >= least, (n_grid, batch, n, fine)
''')


def test_triple_sums_take_whole_rounds():
    """At most two workgroups per CU of 256, the groups of jobs equally often."""
    stub_common.run('''
import numpy as np
for n_grid, n_bins, groups in ((160, 48, 1), (180, 56, 2), (256, 84, 3), (320, 100, 5), (360, 110, 6), (400, 128, 8), (480, 150, 13)):
    a, b, c = np.meshgrid(*[np.arange(1, n_bins + 1, dtype=np.int32)] * 3, indexing="ij")
    tri = np.ascontiguousarray(np.stack([v[(b <= a) & (c <= b) & (c >= a - b)] for v in (a, b, c)], 1))
    h = handle(n_grid, 4, 1, 1, 1000)
    lib.estimator_deposit(h, FAKE, 0, None, 1000)
    lib.estimator_transform(h)
    size = lib.estimator_bispectrum_workspace_bytes(h, 1, n_bins, len(tri))
    ws = np.empty(size + 256, np.uint8)  # not touched but where the job lists go
    at = (ws.ctypes.data + 255) // 256 * 256
    stub.stub_reset(-1)
    lib.estimator_bispectrum(h, 0, 1, n_bins, tri, len(tri), at, size, FAKE, FAKE)
    grids = {stub.stub_grid(i, 0) for i, name in enumerate(launched()) if "k_bs_triple" in name}
    assert len(grids) == 1
    grid = grids.pop()
    assert grid <= 512 and grid % groups == 0 and grid > 512 - groups, (n_grid, n_bins, grid)
    lib.estimator_destroy(h)
''')
