"""The choice of kernel and block shape (csrc/choose.h) against what was measured on MI355X: at each of these sizes the named choice
was the faster one, by the figures beside the rules.  Sizes on both sides of every line."""
import pytest

import choose

V = 128256


def list_kernel(M, d, batch, cap, dense=False, rows=V):
    if choose.wide_supported(rows, M, d, batch, cap, dense):
        return choose.rows_by_hidden(choose.wide_shape(M, d, batch, cap, dense))
    return "head.hip"


@pytest.mark.parametrize("M,d,batch,cap,want", [
    # one sequence, few hidden rows: fewer live rows than capacity
    (8, 4096, 1, 8192, "head.hip"), (8, 4096, 1, 9216, "head.hip"), (8, 4096, 1, 16384, "32x16"), (1, 4096, 1, 8192, "head.hip"), (1, 4096, 1, 16384, "head.hip"),
    (1, 4096, 1, 40960, "32x16"), (8, 2048, 1, 8192, "head.hip"), (8, 1024, 1, 8192, "head.hip"), (8, 1024, 1, 40960, "32x16"),
    (12, 4096, 1, 9216, "32x16"), (12, 2048, 1, 9216, "head.hip"), (12, 2048, 1, 16384, "32x16"), (16, 5120, 1, 9216, "head.hip"), (16, 5120, 1, 32768, "32x16"),
    (16, 8192, 1, 65536, "head.hip"), (1, 8192, 1, 147456, "head.hip"), (1, 4096, 1, 147456, "64x16"),
    # several
    (8, 1024, 4, 9216, "head.hip"), (8, 2048, 4, 9216, "head.hip"), (8, 1024, 8, 9216, "32x16"), (8, 4096, 8, 9216, "32x16"), (8, 4096, 8, 2560, "head.hip"),
    (16, 4096, 2, 5120, "head.hip"), (16, 4096, 2, 9216, "32x16"), (12, 2048, 4, 9216, "head.hip"), (12, 2048, 8, 5120, "32x16"), (16, 4096, 8, 2560, "32x16"),
    (8, 8192, 64, 2560, "64x16"), (8, 8192, 4, 36864, "head.hip"),
])
def test_few_hidden_rows_on_lists(M, d, batch, cap, want):
    assert list_kernel(M, d, batch, cap, rows=200000) == want
