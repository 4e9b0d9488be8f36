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
