"""CPU model of head_hold_kernel (csrc/hold.hip): the rows, columns and LDS words every workgroup touches, over the launchers' own plans.
A list's pieces cover it once, every element index lies inside its buffer, and the choice takes both sides of every line as measured."""
import numpy as np
import pytest

import choose

V = 128256


def pieces(n, np_):
    each, more = n // np_, n % np_
    return [(p * each + min(p, more), p * each + min(p, more) + each + (p < more)) for p in range(np_)]


def check(M, d, batch, cap, n, rows=V, dense=False, pad=4):
    h = choose.hold_plan(d, batch, M, dense)
    MH, col = (M + 3) // 4 * 4, np.arange(64)
    assert 1 <= h.NW <= 8 and 1024 * h.NW >= d > 1024 * (h.NW - 1) and h.lds <= 160 * 1024 and h.parts >= 1 and h.seg % 4 == 0
    lane = (col >> 4) * 32 + (col & 3) * 8
    covered = 0
    for r0, r1 in pieces(n, 8 * h.parts):
        assert r0 == covered
        covered = r1
        if r0 >= r1:
            continue
        nseg = -(-(r1 - r0) // h.seg)
        seg = (-(-(r1 - r0) // nseg) + 3) & ~3
        assert seg <= h.seg
        for s0 in range(r0, r1, seg):
            s1 = min(s0 + seg, r1)
            nq = (s1 - s0 + 3) // 4
            last = (h.NW * MH - 1) * (h.seg + pad) + (nq - 1) * 4 + 3            # the highest partial sum parked
            assert last * 4 < h.lds and s1 <= min(n, cap)
            for i in {0, nq - 1, nq, nq + 3}:                                    # quads past the end are fetched too
                j = np.minimum(s0 + i * 4 + np.arange(4), s1 - 1)
                assert j.min() >= 0 and j.max() < cap
                for w in range(h.NW):
                    for t in range(8):
                        at = w * 1024 + (lane if i < nq else 0) + t * 128
                        at = np.where(w * 1024 + lane + t * 128 < d, at, 0)
                        assert at.max() + 8 <= d and ((rows - 1) * d + at.max() + 8) * 2 <= 2 ** 32
    assert covered == n


@pytest.mark.parametrize("M,d,batch,cap", [(16, 8192, 1, 33344), (5, 8192, 1, 128256), (8, 4096, 64, 5120), (8, 4096, 24, 5120), (1, 2048, 64, 5120), (16, 2568, 3, 5120), (9, 4104, 2, 9216),
                                           (13, 7160, 5, 1600), (8, 2048, 1, 16384), (8, 4096, 256, 1024), (1, 3584, 1, 12288), (4, 8192, 64, 9216)])
def test_pieces_and_addresses(M, d, batch, cap):
    assert choose.hold_supported(V, M, d, batch, cap)
    for n in (0, 1, 7, 8 * choose.hold_plan(d, batch, M).parts + 1, cap // 3, cap):
        check(M, d, batch, cap, n)


@pytest.mark.parametrize("M,d,rows", [(16, 8192, 128256), (9, 4096, 16400)])
def test_dense_heads(M, d, rows):
    assert choose.hold_supported(rows, M, d, 1, rows, dense=True)
    check(M, d, 1, rows, rows, rows, dense=True)


def test_a_row_stride_without_room_for_the_segment_is_rejected():
    with pytest.raises(AssertionError):
        check(16, 8192, 1, 128256, 128256, pad=128)


@pytest.mark.parametrize("M,d,batch,cap,want", [
    (16, 8192, 1, 2560, False), (16, 8192, 1, 3072, False), (4, 8192, 1, 33344, False), (8, 5120, 1, 65536, True), (16, 4608, 1, 65536, False), (8, 4096, 1, 4096, False),
    (8, 4096, 1, 5120, False), (16, 3072, 1, 9216, True), (16, 3072, 1, 20032, False), (4, 4096, 1, 5120, True), (4, 4096, 1, 8192, False), (4, 4096, 1, 16384, True),
    (8, 2048, 1, 9216, False), (8, 2048, 1, 16384, True), (16, 2048, 1, 20032, False), (16, 2048, 1, 65536, True), (8, 1536, 1, 128256, False), (17, 4096, 8, 5120, False),
    (8, 8192, 2, 1024, False), (8, 8192, 4, 1024, True), (4, 8192, 24, 5120, False), (4, 8192, 32, 5120, True), (8, 4096, 4, 1024, False), (8, 4096, 8, 1024, True), (4, 2560, 2, 5120, False),
    (16, 4608, 64, 5120, False), (16, 4608, 16, 5120, True), (8, 2048, 2, 5120, False), (8, 2048, 16, 1024, True), (16, 2048, 8, 5120, False), (16, 2048, 16, 5120, True), (8, 16384, 64, 5120, False),
    (16, 8192, 1, 5120, False), (16, 8192, 1, 5184, True), (16, 4608, 1, 8128, False), (16, 4608, 1, 8192, True), (16, 4608, 1, 32704, True), (16, 4608, 1, 32768, False), (8, 8192, 1, 5120, False), (8, 8192, 1, 5184, True), (8, 4096, 1, 5184, True), (8, 3072, 1, 4160, True), (16, 2560, 1, 9152, True), (16, 2560, 1, 9216, False), (12, 2560, 1, 9216, True), (16, 3072, 1, 12288, True),
    (8, 4096, 11, 5120, True), (8, 4096, 11, 10240, True), (8, 4096, 18, 6080, True), (8, 4096, 18, 6144, True), (8, 4096, 22, 8128, True), (8, 4096, 22, 8192, True), (8, 4096, 32, 704, True), (8, 4096, 32, 768, True), (8, 4096, 33, 4032, True), (8, 4096, 33, 4096, True), (8, 4096, 64, 960, True), (8, 4096, 64, 1024, True), (12, 4096, 64, 5120, True), (16, 4096, 64, 5120, True), (12, 4096, 40, 5120, True),
    (8, 2560, 12, 1984, True), (8, 2560, 12, 2048, True), (8, 4608, 24, 5120, True), (8, 4608, 24, 5504, True), (8, 4096, 24, 8192, True), (1, 4608, 8, 5120, True), (1, 5120, 8, 5120, True), (1, 5120, 4, 5120, True), (1, 5120, 34, 5120, True), (16, 2560, 8, 448, False), (16, 2560, 8, 512, False), (8, 5120, 8, 960, True), (8, 5120, 8, 1024, True), (4, 4096, 8, 960, True), (4, 4096, 8, 1024, True), (4, 3072, 8, 2048, True), (4, 3072, 8, 2560, True), (8, 2048, 3, 8192, True), (16, 5120, 1, 5184, True), (16, 8192, 4, 2048, True),
])
def test_choice(M, d, batch, cap, want):
    assert choose.hold_supported(V, M, d, batch, cap) == want


def test_workgroups():
    plan = lambda d, batch, dense=False: choose.hold_plan(d, batch, 8, dense).parts * 8 * batch
    assert plan(8192, 1) == plan(2048, 1) == 256 and plan(4096, 32) == 256 and plan(4096, 64) == 512 and plan(4096, 48) == 768 and plan(4096, 24) == 192
    assert plan(4096, 20) == 480 and plan(2048, 16) == 512 and plan(4096, 256) == 2048 and plan(4096, 1, True) == 512 and plan(8192, 1, True) == 1024
