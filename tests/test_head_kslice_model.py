"""CPU model of head_kslice_kernel (csrc/kslice.hip): rows, hidden rows, columns and LDS bytes of every block over the launchers' own plans.  Every (row, hidden row)
pair is covered once, every fetch and every fragment read lies inside its buffer, and the wait before a slot is read covers its own fetches and no younger ones."""
import numpy as np
import pytest

import choose

V = 128256


def slots(L):
    return 4 if L <= 4 else 3 if L <= 6 else 2


def lds_bytes(LB, rows):
    sizes = [la for la in range(1, rows // 8 + 1) if la != 7]
    return max(max(4 * slots(la + LB) * (la + LB) * 1024 + 1024, 4 * 16 * ((LB + 1) // 2) * (16 * ((la + 1) // 2) + 4) * 4) for la in sizes)


def rows_of(block):
    la = -(-block // 8)
    return 8 if la == 7 else la


def check_block(rows, most, LB, M, d, m0, waits=lambda R, L: (R - 1) * L):
    LA = rows_of(rows)
    L, FR, FH = LA + LB, (LA + 1) // 2, (LB + 1) // 2
    R, lds = slots(L), lds_bytes(LB, most)
    assert rows <= 8 * LA <= most and waits(R, L) <= 63
    nk, lane = -(-d // 64), np.arange(64)
    seen = []
    for w in range(4):
        mine = -(-(nk - w) // 4) if nk > w else 0
        for i in range(mine):
            k0 = (w + i * 4) * 64
            c = ((lane & 7) ^ (lane >> 3)) * 8
            at = k0 + c if k0 + 64 <= d else np.where(k0 + c < d, c + k0, 0)
            assert at.min() >= 0 and at.max() + 8 <= d
        seen += [w + i * 4 for i in range(mine)]
        issued = min(R, mine)                                           # steps fetched when step 0 is waited for
        for i in range(mine):
            left = waits(R, L) if i + R <= mine else 0
            assert issued * L - left >= (i + 1) * L, "the slot's own fetches have landed"
            issued += i + R < mine
        assert issued == mine
        for base in (0, LA * 1024):                                     # fragment reads of the wavefront's last slot
            for frag in range(FR if base == 0 else FH):
                for kk in (0, 1):
                    at = (w * R + R - 1) * L * 1024 + base + frag * 2048 + (lane & 15) * 128 + (((lane >> 4) + 4 * kk) ^ (lane & 7)) * 16
                    assert at.max() + 16 <= lds
                    for grp in range(0, 64, 8):                          # eight lanes of a 128-byte access: all banks different
                        assert len(set((at[grp:grp + 8] // 16 % 8).tolist())) == 8
    assert sorted(seen) == list(range(nk))
    assert 4 * 16 * FH * (16 * FR + 4) * 4 <= lds <= 160 * 1024
    assert m0 < M


def check(M, d, batch, cap, n):
    plan = choose.kslice_plan(M, batch, cap)
    assert plan.LB in (2, 3, 4, 5, 6, 8) and plan.hid_blocks == -(-M // (8 * plan.LB)) and plan.parts >= 1
    assert plan.rows % 8 == 0 and 8 <= plan.rows <= 64 and plan.rows != 56
    grid = 8 * plan.parts * plan.hid_blocks * batch
    assert grid < 262144
    pieces, np_ = {}, 8 * plan.parts
    over = lambda n, x: n if x == 1 else n * (-(-2 ** 32 // x)) >> 32
    for v in (n, cap, 262144):
        assert over(v, np_) == v // np_
    for blk in range(grid):
        x, xr = blk & 7, blk >> 3
        y = over(xr, plan.hid_blocks)
        hb, part = xr - y * plan.hid_blocks, over(y, batch)
        if y - part * batch == 0:
            assert part < plan.parts and (x * plan.parts + part, hb) not in pieces
            pieces[x * plan.parts + part, hb] = 1
    assert len(pieces) == np_ * plan.hid_blocks
    each, more, covered, kinds = n // np_, n % np_, 0, set()
    for p in range(np_):
        r0 = p * each + min(p, more)
        r1 = r0 + each + (p < more)
        assert r0 == covered
        covered = r1
        if r1 > r0:
            nseg = -(-(r1 - r0) // plan.rows)
            seg = -(-(r1 - r0) // nseg)
            for j0 in range(r0, r1, seg):
                assert 0 < min(j0 + seg, r1) - j0 <= plan.rows and min(j0 + seg, r1) <= cap
                kinds.add(min(j0 + seg, r1) - j0)
    assert covered == n
    for rows in kinds:
        for hb in range(plan.hid_blocks):
            check_block(rows, plan.rows, plan.LB, M, d, hb * 8 * plan.LB)


@pytest.mark.parametrize("M,d,batch,cap", [(64, 3584, 1, 4352), (17, 512, 1, 3072), (33, 1032, 1, 16384), (40, 8192, 1, 20480), (24, 4096, 16, 1792), (64, 4096, 3, 2048), (60, 2056, 8, 2880), (48, 1024, 2, 1000),
                                           (20, 3000, 13, 640)])
def test_pieces_and_addresses(M, d, batch, cap):
    assert choose.kslice_supported(V, M, d, batch, cap)
    for n in (0, 1, 9, cap // 5, cap * 4 // 7 - 1, cap * 4 // 7, cap):
        check(M, d, batch, cap, n)


def test_every_block():
    for LB in (2, 3, 4, 5, 6, 8):
        for rows in range(1, 65):
            for most in {64, 64 if rows > 48 else -(-rows // 8) * 8}:
                check_block(rows, most, LB, 8 * LB, 72, 0)
                check_block(rows, most, LB, 8 * LB, 1096, 0)


def test_a_wait_for_a_younger_step_only_is_rejected():
    with pytest.raises(AssertionError):
        check_block(24, 24, 4, 32, 1096, 0, waits=lambda R, L: R * L)


@pytest.mark.parametrize("M,d,batch,cap,want", [
    (64, 3584, 1, 4352, True), (64, 3584, 1, 33344, False), (40, 3584, 1, 33344, False), (20, 3584, 1, 33344, False), (20, 4096, 1, 65536, False), (20, 4096, 1, 128256, False), (64, 2048, 1, 20480, True), (64, 2048, 1, 33344, False),
    (32, 2048, 1, 33344, False), (32, 1024, 1, 20480, True), (32, 1024, 1, 33344, False), (64, 512, 1, 2624, True), (32, 512, 1, 8192, False), (16, 4096, 1, 4352, False), (65, 4096, 1, 4352, False), (32, 504, 1, 640, False),
    (64, 4096, 4, 5120, True), (20, 4096, 16, 5120, False), (32, 4096, 16, 1920, False), (48, 4096, 16, 2048, False), (20, 4096, 12, 1024, False), (20, 4096, 24, 1024, False), (64, 1024, 4, 5120, False), (20, 1024, 16, 1024, True),
    (60, 4096, 8, 4032, False), (60, 4096, 8, 2880, True),
    (20, 3584, 1, 24576, True), (20, 3584, 1, 24640, False), (32, 3584, 1, 32768, True), (32, 3584, 1, 32832, False), (40, 3584, 1, 20480, True), (40, 3584, 1, 20544, False), (48, 1024, 1, 16384, True), (48, 1024, 1, 16448, False), (64, 1024, 1, 8192, True), (64, 1024, 1, 8256, False), (32, 2048, 1, 20480, True), (32, 2048, 1, 20544, False),
    (17, 8192, 1, 960, False), (17, 8192, 1, 1024, True), (33, 8192, 1, 960, False), (33, 8192, 1, 1024, True), (24, 7168, 1, 960, False), (24, 7168, 1, 1024, True), (33, 7168, 1, 320, True), (17, 6144, 1, 320, True), (64, 4096, 14, 960, False), (64, 4096, 14, 1024, True), (48, 4096, 14, 384, False), (48, 4096, 14, 448, True), (32, 4096, 14, 320, True), (20, 8192, 4, 384, False), (20, 8192, 4, 448, True), (64, 2048, 2, 10240, True), (64, 2048, 2, 10304, False), (20, 2048, 2, 14336, True), (20, 4096, 16, 1792, True), (20, 4096, 16, 1856, False),
])
def test_choice(M, d, batch, cap, want):
    assert choose.kslice_supported(V, M, d, batch, cap) == want
    assert not choose.kslice_supported(V, M, d, batch, cap, aligned=False) and not choose.kslice_supported(V, M, d, 1, V, dense=True)
