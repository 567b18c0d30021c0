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


@pytest.mark.parametrize("M,d,rows,want", [
    (1, 512, 128256, "64x16"), (4, 512, 16400, "head.hip"), (1, 1024, 128256, "head.hip"), (16, 768, 128256, "head.hip"),
    (9, 2048, 50001, "head.hip"), (16, 2048, 16400, "head.hip"), (9, 4096, 128256, "head.hip"), (16, 4096, 128256, "64x16"), (16, 4096, 16400, "head.hip"),
    (9, 2560, 16400, "64x16"), (16, 3584, 128256, "64x16"), (16, 5120, 128256, "64x16"), (16, 6144, 128256, "head.hip"), (16, 8192, 128256, "head.hip"),
    (8, 2048, 128256, "head.hip"), (8, 2560, 128256, "64x16"), (5, 3072, 50001, "head.hip"), (8, 3584, 128256, "head.hip"), (8, 4096, 128256, "head.hip"),
    (8, 5120, 128256, "64x16"), (8, 5120, 16400, "head.hip"), (4, 2048, 128256, "head.hip"),
    (16, 1024, 128256, "64x16"), (8, 1024, 128256, "head.hip"), (16, 512, 24000, "64x16"), (16, 3584, 24000, "64x16"), (9, 3584, 20480, "head.hip"),
])
def test_few_hidden_rows_dense(M, d, rows, want):
    assert list_kernel(M, d, 1, rows, dense=True, rows=rows) == want


def test_loads_per_wavefront():
    assert choose.quad_plan(4, 2048, 1, 128256, dense=True).KS == 8 and choose.quad_plan(4, 2048, 1, 50001, dense=True).KS == 4
    assert choose.quad_plan(4, 1536, 1, 128256, dense=True).KS == 4 and choose.quad_plan(8, 2048, 1, 128256, dense=True).KS == 4
    assert choose.quad_plan(4, 2048, 1, 8192).KS == 4 and choose.quad_plan(4, 1024, 1, 8192).KS == 2 and choose.quad_plan(4, 2056, 1, 8192).KS == 8


@pytest.mark.parametrize("M,d,batch,cap,want", [
    (17, 2048, 1, 1088, "head.hip"), (17, 1792, 1, 1088, "32x32"), (33, 2048, 1, 1088, "32x32"), (32, 2048, 2, 2560, "32x32"), (32, 4096, 1, 4352, "32x32"),
    (64, 4096, 1, 2560, "32x32"), (64, 4096, 1, 2496, "head.hip"), (17, 4096, 2, 2560, "32x32"), (17, 8192, 2, 2560, "head.hip"), (17, 8192, 2, 5120, "32x32"),
    (33, 4096, 2, 2560, "head.hip"), (33, 4096, 8, 1088, "32x32"), (64, 4096, 2, 2560, "32x32"), (33, 4096, 8, 320, "head.hip"), (33, 8192, 8, 1088, "head.hip"),
    (64, 8192, 8, 1088, "32x32"), (64, 8192, 2, 2560, "head.hip"), (17, 8192, 2, 9216, "32x32"), (64, 4096, 2, 5120, "32x64"), (60, 4096, 8, 4096, "64x64"),
    (70, 4096, 2, 2560, "32x32"), (130, 8192, 2, 3072, "32x32"), (17, 12288, 2, 2560, "32x32"),
])
def test_17_to_64_hidden_rows_on_lists(M, d, batch, cap, want):
    assert list_kernel(M, d, batch, cap) == want


@pytest.mark.parametrize("M,rows,dense,want", [
    (70, 16448, False, "64x64"), (70, 32768, False, "64x64"), (128, 49152, False, "256x128"), (128, 98240, False, "256x128"), (130, 24576, False, "64x64"),
    (130, 49152, False, "gemm"), (256, 24576, False, "64x64"), (256, 32768, False, "gemm"), (512, 16448, False, "gemm"), (512, 98240, False, "gemm"),
    (65, 24000, True, "64x64"), (128, 36000, True, "256x128"), (200, 20480, True, "64x64"), (128, 50001, True, "256x128"), (129, 16400, True, "64x64"), (200, 24000, True, "gemm"), (512, 16400, True, "gemm"), (1024, 24000, True, "gemm"),
    (64, 24000, True, "128x64"), (33, 16384, True, "128x64"), (64, 12000, True, "64x64"),
])
def test_shapes_for_many_hidden_rows(M, rows, dense, want):
    assert list_kernel(M, 4096, 1, rows, dense=dense, rows=rows) == want
    assert choose.rows_by_hidden(choose.wide_shape(M, 4096, 1, rows, dense, aligned=False)) == want.replace("gemm", "256x256")
    assert choose.rows_by_hidden(choose.wide_shape(M, 4104, 1, rows, dense)) == want.replace("gemm", "256x256")


@pytest.mark.parametrize("batch,window,longest,want", [
    (1, 256, 256, True), (1, 640, 600, True), (1, 1024, 600, False), (1, 4096, 331, True), (1, 8192, 64, True), (1, 8192, 500, False), (1, 16384, 0, False), (1, 235312, 64, False),
    (16, 512, 512, True), (16, 16384, 64, False), (64, 1024, 1024, True), (64, 8192, 600, True), (64, 8192, 1500, False), (64, 65536, 64, False), (64, 235312, 64, False),
])
def test_stream_initialisation(batch, window, longest, want):
    """a short prompt for a wide window may follow a stream that filled it, and one workgroup would undo it token by token"""
    assert choose.vocab_init_serial(batch, window, longest) == want


def test_selection_in_chunks():
    assert choose.topk_chunks(8, 10, topk_cap=65000) and choose.topk_chunks(8, 10, topk_cap=1, window=30000, distinct=True)     # lists that fill their room
    assert choose.topk_chunks(16, 10, topk_cap=1, window=235312) and not choose.topk_chunks(16, 10, topk_cap=1, window=33303)    # windows of raw tokens
    assert not choose.topk_chunks(8, 10, topk_cap=4000, window=13000) and not choose.topk_chunks(88, 10, topk_cap=65000)
    assert not choose.topk_chunks(8, 40, topk_cap=32000) and choose.topk_chunks(8, 40, topk_cap=128000)
    assert choose.topk_chunks(95, 40, dense=True) and not choose.topk_chunks(96, 1, dense=True)


def test_batch_union_head():
    assert not choose.union_feeds(16, 2496) and choose.union_feeds(16, 2560)
    assert not choose.union_split_pairs(40959, 0) and choose.union_split_pairs(40960, 3200) and not choose.union_split_pairs(40960, 3201)        # 40 000 pairs: a thirteenth
    assert choose.union_split_pairs(131072, 32768) and not choose.union_split_pairs(131072, 32769)                                            # 131 072: a quarter
    assert choose.union_split_pairs(196608, 73728) and not choose.union_split_pairs(1 << 26, (1 << 26) * 3 // 8 + 1) and choose.union_split_pairs(1 << 26, (1 << 26) * 3 // 8)
