"""Which rows the units of an aggregation launch take, on the host: every row once per column
workgroup, none outside the matrix, for operands far taller than a test could hold."""
import ctypes as C

import numpy as np
import pytest

q = pytest.importorskip("paper_2111_09547_amd")
import paper_2111_09547_amd.binding as b  # noqa: E402


def units(rows, cols, block_rows, x_cols, out_cols):
    d, _ = b.describe(rows, cols, 1, b.LEFT, block_rows)
    d.data = 0x10000                                 # never read
    probe = b.lib().qgtc_probe_units
    n = probe(C.byref(d), x_cols, out_cols, 0, 0, *[np.zeros(1, np.int32).ctypes.data] * 3)
    assert n > 0
    col, row0, here = (np.zeros((n, 4), np.int32) for _ in range(3))
    assert probe(C.byref(d), x_cols, out_cols, 0, n, col.ctypes.data, row0.ctypes.data, here.ctypes.data) == n
    return col, row0, here


@pytest.mark.parametrize("rows,cols,block_rows,x_cols,out_cols", [
    # tall operands: more workgroups than 2^32 / (their number) allows without a correction
    (16_777_372, 128, 0, 16, 0), (33_000_000, 128, 0, 16, 0), (11_900_001, 128, 0, 128, 0),
    (8_470_123, 128, 0, 256, 0), (16_777_372, 128, 0, 16, 16), (33_000_001, 96, 0, 100, 64),
    (400_000_001, 128, 0, 16, 0),
    # one tall diagonal block and a part of a second, and many small ones
    (17_000_033, 16_777_408, 16_777_408, 16, 0), (5_000_000, 96, 96, 48, 0), (5_000_000, 32, 32, 16, 16),
    # ordinary ones
    (1, 128, 0, 16, 0), (63, 64, 0, 33, 0), (8192, 8192, 0, 64, 0), (65536, 1024, 1024, 128, 64),
    (15221, 416, 416, 300, 101), (262144, 2048, 2048, 512, 16), (1000, 128, 128, 20, 7),
])
def test_every_row_is_taken_once(rows, cols, block_rows, x_cols, out_cols):
    col, row0, here = units(rows, cols, block_rows, x_cols, out_cols)
    on = here > 0
    assert (row0[on] >= 0).all() and (row0[on].astype(np.int64) + here[on] <= rows).all()
    n_col = int(col.max()) + 1
    first = np.sort(row0[on])
    order = np.argsort(row0[on], kind="stable")
    starts, lens = row0[on][order][::n_col].astype(np.int64), here[on][order][::n_col]
    assert (np.bincount(col[on]) == len(starts)).all()           # the same rows along every column workgroup
    assert (first.reshape(-1, n_col) == first.reshape(-1, n_col)[:, :1]).all()
    assert starts[0] == 0 and (starts[1:] == starts[:-1] + lens[:-1]).all() and starts[-1] + lens[-1] == rows


@pytest.mark.parametrize("x_cols,out_cols", [(5, 0), (40, 0), (5, 7), (200, 7)])
def test_rows_of_up_to_128_MiB(x_cols, out_cols):
    """Rows far apart are taken like those side by side; at 2^25 words they are refused."""
    for ld, taken in (((1 << 24) - 4, True), (1 << 24, True), ((1 << 25) - 4, True), (1 << 25, False)):
        d, _ = b.describe(70, 300, 1, b.LEFT)
        d.data, d.ld_words = 0x10000, ld
        out = [np.zeros((4, 4), np.int32) for _ in range(3)]
        n = b.lib().qgtc_probe_units(C.byref(d), x_cols, out_cols, 0, 4, *[o.ctypes.data for o in out])
        assert (n > 0) == taken, ld
        if taken:
            assert sorted(set(out[1][out[2] > 0].tolist())) == [0, 64] and out[2].max() == 64
