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
