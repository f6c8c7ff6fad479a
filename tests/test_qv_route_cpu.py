"""The rule that picks the windowed route of the overlaps (a host function of the
library): only where its launches fit a grid, since the automatic route has to
give way to the next one otherwise."""
import ctypes as C
import os

import pytest

import paper_2505_11655_amd as ile


@pytest.fixture(scope="module")
def win_ok():
    if not os.path.exists(ile.LIB_PATH):
        pytest.skip("libile.so not built")
    # ile::qv_win_ok(int64_t n, int64_t n_band, int64_t cols, int n_time)
    f = C.CDLL(ile.LIB_PATH)._ZN3ile9qv_win_okEllli
    f.argtypes, f.restype = [C.c_int64, C.c_int64, C.c_int64, C.c_int], C.c_bool
    return f


@pytest.mark.parametrize("n,n_band,cols,n_time,ok", [
    (16384, 8034, 6912, 410, True),                       # the event grid
    (16400, 8034, 6912, 410, False),                      # no multiple of 512
    (16384, 160, 6912, 410, False),                       # a narrow band: the direct sum is cheaper
    (1 << 31, 1 << 30, 27, 410, False),                   # 32-bit indices of the grid
    (512, 512, (1 << 31) - 1, 1, True), (512, 512, 1 << 31, 1, False),                  # blocks of one launch
    (512, 512, 1 << 30, 512, True), (1024, 1024, 1 << 30, 1024, False),                 # two window blocks a column
    (1 << 25, 1 << 25, 1, 65535 * 512, True), (1 << 26, 1 << 26, 1, 65536 * 512, False),   # window blocks in the grid's z
])
def test_windowed_route_rule(win_ok, n, n_band, cols, n_time, ok):
    assert win_ok(n, n_band, cols, n_time) == ok
