"""Host work of repeated calls (CPU, on the stub)."""

import pytest

import stub_common

pytest.importorskip("paper_1512_07295_amd", reason="libfsest.so not built")


def test_occupancy_is_asked_once_per_handle():
    stub_common.run('''
def calls(h):
    lib.estimator_deposit(h, FAKE, 0, None, 5000)
    lib.estimator_transform(h)
    lib.estimator_power(h, 1, 8, 0, FAKE, FAKE, FAKE)
    lib.estimator_export_delta(h, 0, FAKE)
    lib.estimator_power(h, 1, 8, 0, FAKE, FAKE, FAKE)  # of the stored spectrum
    lib.estimator_backward(h, FAKE, 0, None, 5000, FAKE, 1, 8, FAKE)

for n_grid in (32, 60):
    for code in range(4):
        h = handle(n_grid, 4, code)
        stub.stub_reset(-1)
        calls(h)
        first = stub.stub_occupancy_queries()
        assert 0 < first <= 3
        blocks = [(name, stub.stub_grid(i, 0)) for i, name in enumerate(launched())]
        stub.stub_reset(-1)
        for _ in range(5):
            calls(h)
        assert stub.stub_occupancy_queries() == 0, (n_grid, code)
        assert {(name, stub.stub_grid(i, 0)) for i, name in enumerate(launched())} <= set(blocks)
        lib.estimator_set_launch(h, 35)  # the defaults
        calls(h)
        assert stub.stub_occupancy_queries() == 0
        lib.estimator_destroy(h)
''')


def test_autotune_tries_what_the_call_reads():
    """The stub's times fall from trial to trial, so that every parameter that is
    tried changes and the others keep their defaults (choice 35)."""
    stub_common.run('''
def digits(choice):
    return choice // 24, choice // 8 % 3, choice // 4 % 2, choice // 2 % 2, choice % 2

# (n_grid, order, interlace, particles): tried lines, reduction, deposit
for n_grid, order, code, n, tried in ((32, 4, 1, 5000, (1, 1, 0)), (60, 4, 1, 5000, (0, 1, 0)), (32, 4, 2, 5000, (1, 0, 0)),
                                      (100, 3, 3, 5000, (0, 0, 0)), (32, 5, 1, 5000, (1, 1, 1)), (16, 2, 0, 500, (1, 1, 1)),
                                      (512, 2, 1, 1 << 20, (1, 1, 1)), (512, 2, 1, 1 << 26, (1, 1, 0))):
    h = handle(n_grid, order, code, 1, n)
    got = digits(lib.estimator_autotune(h, FAKE, 0, None, n, 1, 4, 1))
    default = digits(35)
    for i, on in ((0, tried[0]), (1, tried[1]), (2, tried[2]), (3, 0), (4, tried[2])):
        assert (got[i] != default[i]) == bool(on), (n_grid, order, code, n, got)
    lib.estimator_destroy(h)
''')
