"""CPU model of the address arithmetic of the kernels that load without bounds tests.

The head and the selection have kernels whose loads are unconditional: instead of testing every address they clamp rows and
columns into range and mask by arithmetic (csrc/head.hip: head_quad_kernel with row groups of four,
head_quad_private_kernel<FAST>, head_tile64_kernel<FAST 1 / 2>; csrc/wide.hip: head_wide_kernel, head_gemm_kernel; csrc/topk.hip: the
shifted loads of unaligned rows and the walk in 16-byte pieces).  Whether that is safe depends on which one the
launcher picks for which shape.  The choice is the launchers' own (csrc/choose.h, compiled for the CPU); this file restates, in plain Python, the
control flow around it and every element index the lanes form for H [batch][M][d], W [V][d], the id list [batch][cap], the row counts
[batch], the columns [batch][cap] and the logits [batch][M][ld] (or the split-K planes), and asserts that all of them lie inside their
buffers, that every block of live logits is computed once, that operands kept in LDS are read where they were put, and -- where fetches
are counted instead of waited for one by one -- that no piece of LDS is read before it has landed or refilled before it has been read.
A variant choice that once faulted on the GPU (constant hidden-row strides
taken with M = 32: wavefronts 2-3 addressed hidden rows 32..63 past the end of H) must be rejected by the model, and so must a planted
mistake of every other kind.  New unconditional-load variants go through this model before they go to the GPU."""
import functools
import itertools
import os
import re

import numpy as np
import pytest

import choose


class OutOfBounds(AssertionError):
    pass


def need(cond, *what):
    if not cond:
        raise OutOfBounds(what)


def ceil_div(a, b):
    return (a + b - 1) // b


# ---- the launchers' control flow (launch_head, launch_head_64) ---------------------------------------------------------
def plan(V, M, d, batch, cap, dense, partial_bytes=1 << 62, aligned=True):
    """list of (kernel, params, first hidden row, hidden rows) one launch_head call uses"""
    if choose.wide_supported(V, M, d, batch, cap, dense):
        shape = choose.wide_shape(M, d, batch, cap, dense, aligned)
        if shape == choose.GEMM:
            return [("gemm", {}, 0, M)]
        return [("wide", dict(shape=shape, by_die=choose.wide_by_die(M, batch, cap, dense)), 0, M)]
    if M > 64:
        if batch > 1:
            return [("generic", {}, 0, M)]                          # one wavefront per row, every load tested
        return [(k, p, m0, mm) for m0 in range(0, M, 64) for k, p, _, mm in plan_64(min(64, M - m0), d, 1, cap, dense, partial_bytes)]
    return plan_64(M, d, batch, cap, dense, partial_bytes)


def plan_64(M, d, batch, cap, dense, partial_bytes):
    if M <= 16:
        q = choose.quad_plan(M, d, batch, cap, dense)
        if q.loop:
            need(q.KS == (8 if q.MT <= 2 else 4), "instantiations with a K loop")
            return [("private", dict(RT=q.RT, MT=q.MT, KS=q.KS, NW=4, fast=d % (4 * 128 * q.KS) == 0), 0, M)]
        return [("quad", dict(NRG=q.NRG, RT=q.RT, MT=q.MT, KS=q.KS), 0, M)]
    S = ceil_div(d, 512)
    split = choose.head_split(M, d, batch, cap, dense, partial_bytes, cap)
    return [("tile64", dict(MT=2 if M <= 32 else 4, fast=choose.tile64_fast(M, d), split=split, S=S), 0, M)]


# ---- the kernels' index arithmetic -------------------------------------------------------------------------------------
LANES = np.arange(64)
OROW, PART, Q = (LANES & 15) >> 2, LANES & 3, LANES >> 4


def check_quad(M, d, batch, cap, V, n, dense, NRG, RT, MT, KS, ld=None):
    ld = ld or (V if dense else cap)
    ROWS, RPG = 4 * RT * NRG, 4 * RT
    need(d <= 512 * KS and M <= 4 * MT, "quad needs one K-iteration and a row tile per four hidden rows")
    need(4 * MT * KS * 1024 + 4 * NRG * RT * MT * 16 * 4 <= 160 * 1024 and RT * MT * 16 <= 256, "LDS, one output per thread")
    tiles = ceil_div(cap, ROWS)
    uncond = RT == 1
    HI = MT * KS
    HPW = ceil_div(HI, NRG)
    seen = np.zeros(d, bool)
    for kq in range(4):
        for t in range(KS):
            c = (kq * 128 * KS + Q * 32 + PART * 8 + t * 128)[(LANES & 15) < 4]
            for cc in c[c < d]:
                need(not seen[cc:cc + 8].any(), "column twice", cc)
                seen[cc:cc + 8] = True
    need(seen.all(), "every column once", d, KS)
    for b in (0, batch - 1):
        for tile in (0, tiles - 1):
            for w in range(4 * NRG):
                kq, rg = w & 3, w >> 2
                j0 = (tile * NRG + rg) * RPG
                if not dense:                                   # int4 loads of the ids, not waiting for n
                    need(j0 + 4 * RT <= cap, "ids", j0, cap)
                coff = kq * 128 * KS + Q * 32 + PART * 8
                for ii in range(HPW):
                    i = rg * HPW + ii
                    if uncond:
                        ic = min(i, HI - 1)
                        mt, t = ic // KS, ic % KS
                        m = np.minimum(mt * 4 + OROW, M - 1)
                        c = coff + t * 128
                        c = np.where(c < d, c, 0)
                        need(np.all((m >= 0) & (m < M)) and np.all(c + 8 <= d), "H", M, d, i)
                    # the predicated form tests i < HI, m < M, c < d before it loads
                live = j0 < n
                for t in range(KS):
                    c = coff + t * 128
                    if uncond:
                        c = np.where(live & (c < d), c, 0)
                        need(np.all(c + 8 <= d), "W col", d, t)  # rows are clamped into [0, V) or replaced by row 0
                # stores: j < n and m < M
                need(n <= cap <= ld or dense, "logit row stride")


def check_private(M, d, batch, cap, V, n, dense, RT, MT, KS, NW, fast):
    ROWS = 4 * RT
    tiles = ceil_div(cap, ROWS)
    if not dense:
        need(tiles * ROWS <= cap, "ids", cap, ROWS)             # int4 loads j0 .. j0 + 4*RT
    if not fast:
        return                                                  # the generic form tests c < d and m < M per load
    need(d % (NW * 128 * KS) == 0, "FAST needs whole K-iterations")
    for kb in range(0, d, NW * 128 * KS):
        for w in range(NW):
            coff = w * 128 * KS + Q * 32 + PART * 8
            for t in range(KS):
                need(np.all(kb + coff + t * 128 + 8 <= d), "col", d, kb, w, t)
    for mt in range(MT):
        m = np.minimum(mt * 4 + OROW, M - 1)
        need(np.all((m >= 0) & (m < M)), "H row")


def check_tile64(M, d, batch, cap, V, n, dense, MT, fast, split, S, partial_elems=None):
    if not dense:
        need(ceil_div(cap, 64) * 64 <= cap, "ids: one per lane up to the tile's end", cap)
    if fast:
        need(d % 512 == 0, "FAST needs whole slices")
        for sl in range(S):
            need(np.all(sl * 512 + LANES * 8 + 8 <= d), "col")
        for b in range(batch):
            for w in range(4):
                for r in range(16):
                    m = w * 16 + r
                    if fast == 1:
                        m = min(m, M - 1)
                    need(0 <= b * M + m < batch * M if fast == 1 else b * M + m < (b + 1) * M, "H row", M, w, r)
    if split:
        need(cap % 64 == 0 and cap % 4 == 0, "plane rows")
        # every live tile stores four consecutive logits per lane without looking at n: j0 + 15 < cap
        need(ceil_div(cap, 64) * 64 <= cap, "plane store")
        if partial_elems is not None:
            need(S * batch * M * cap <= partial_elems, "planes", S, batch, M, cap)


def check_wide_steps(d, BK, D, tail, CPR, parity=None):
    """the K walk of head_wide_kernel: which step's columns each register set and LDS stage holds when it is multiplied"""
    nk = ceil_div(d, BK)
    held = [min(j, nk - 1) for j in range(D)]                    # step in each register set
    stage = [held[0], None]
    done = []
    for ks in range(0, nk, D):
        for j in range(D):
            st = ks + j
            held[j] = min(st + D, nk - 1)
            if (D == 2 and not tail) or st < nk:
                need(stage[j & 1] == st, "stage holds the step that is multiplied", d, BK, D, st, stage)
                done.append(st)
            label = min(st + 1, nk - 1) if parity is None else parity(st)
            need(held[(j + 1) % D] == label, "the set that is parked holds the step it is masked as", st)
            stage[(j + 1) & 1] = held[(j + 1) % D]
    need(done == list(range(nk)), "every step once", d, done)
    # columns: piece pc of step ks is column ks * BK + pc * 8; past d it is fetched from column 0 and parked as zeros
    seen = np.zeros(d // 8, int)
    for ks in range(nk):
        pc = np.arange(CPR)
        off = ks * BK * 2 + pc * 16
        if tail:
            off = np.where(off >= d * 2, 0, off)
        need(np.all(off + 16 <= d * 2), "column bytes", d, ks)
        real = ks * BK + pc * 8 < d
        need(np.all(real | (tail and ks * BK + BK > d)), "unmasked columns past d", d, ks)
        seen[(ks * BK + pc * 8)[real] // 8] += 1
    need(np.all(seen == 1), "every column once", d)


def check_wide(M, d, V, n, cap_rows, ld, shape, batch=1, by_die=False, ids_stride=None, opos=False, seq_rows=0, nseq=None, dense=False, tail=None, blocks=None):
    """head_wide_kernel (csrc/wide.hip): BM x BN blocks of logits, K in steps of BK, both operand blocks through LDS.  n: a row count or one per
    sequence."""
    WR, WH, FR, FH, BK, D = blocks or choose.block(shape)
    ns = [n] * batch if np.isscalar(n) else list(n)
    need(choose.wide_reaches(V, M, d), "32-bit byte offsets")
    NT = 64 * WR * WH
    BM, BN = WR * FR * 16, WH * FH * 16
    CPR = BK // 8
    RPP = NT // CPR
    NA, NB = BM // RPP, BN // RPP
    STR = BK * 2 + 32
    STAGE = (BM + BN) * STR
    tail = d % (D * BK) != 0 if tail is None else tail
    need(2 * STAGE <= 160 * 1024 and BM % RPP == 0 and BN % RPP == 0 and D % 2 == 0, "tile shape")
    check_wide_steps(d, BK, D, tail, CPR)
    row_blocks, hid_blocks = ceil_div(cap_rows, BM), ceil_div(M, BN)
    if batch == 1:
        grid = ceil_div(row_blocks, 8) * hid_blocks * 8
    else:
        grid = ceil_div(row_blocks, 8) * hid_blocks * batch * 8 if by_die else row_blocks * hid_blocks * batch
    blk = np.arange(grid, dtype=np.int64)
    nv = np.array(ns, np.int64)
    if batch == 1:
        xq, xr = blk & 7, blk >> 3
        b, hb, rb = np.zeros_like(blk), xr % hid_blocks, (xr // hid_blocks) * 8 + xq
        keep = rb < row_blocks
    else:
        x, xr = blk & 7, (blk >> 3) if by_die else blk
        hb = xr % hid_blocks if by_die else xr // batch % hid_blocks
        b = (xr // hid_blocks if by_die else xr) % batch
        rb = xr // batch // hid_blocks
        keep = np.ones(grid, bool)
        if by_die:
            nb = (nv[b] + BM - 1) // BM
            rb = rb + ((x * nb + (b & 7)) >> 3)
            keep = rb < (((x + 1) * nb + (b & 7)) >> 3)
        keep &= rb < row_blocks
    keep &= rb * BM < nv[b]
    b, hb, rb = b[keep], hb[keep], rb[keep]
    code = (b * row_blocks + rb) * hid_blocks + hb
    need(len(np.unique(code)) == len(code), "a block of logits computed twice")
    need(len(code) == sum(ceil_div(x, BM) for x in ns) * hid_blocks, "every live block of every sequence", len(code), ns, by_die)

    ids_stride = cap_rows if ids_stride is None else ids_stride
    tid = np.arange(NT)
    pc, pr = tid % CPR, tid // CPR
    lane, w = tid & 63, tid >> 6
    wr, wh = w // WH, w % WH
    opos_len = cap_rows // 4 * 4
    for bb, q_rb, q_hb in sorted({(s, r, h) for s in {0, batch // 2, batch - 1} for r in {0, (ns[s] - 1) // BM} for h in (0, hid_blocks - 1) if ns[s]}):
        nn, j0, m0 = ns[bb], q_rb * BM, q_hb * BN
        for i in range(NA):
            j = j0 + pr + i * RPP
            j = np.where(j < nn, j, j0)
            if not dense:
                need(np.all(bb * ids_stride + j < (bb + 1) * ids_stride), "ids", j.max(), ids_stride)
            # rows are clamped into [0, V)
            need(np.all((pr + i * RPP) * STR + pc * 16 + 16 <= BM * STR), "LDS park A")
        for i in range(NB):
            m = np.minimum(m0 + pr + i * RPP, M - 1)
            need(np.all((m >= 0) & (m < M)), "H row")
            need(np.all((pr + i * RPP) * STR + pc * 16 + 16 <= BN * STR), "LDS park B")
        frag = (lane & 15) * STR + (lane >> 4) * 16
        for kk in range(BK // 32):
            need(np.all((wr * FR * 16 + (FR - 1) * 16) * STR + frag + kk * 64 + 16 <= BM * STR), "LDS read A")
            need(np.all(BM * STR + (wh * FH * 16 + (FH - 1) * 16) * STR + frag + kk * 64 + 16 <= STAGE), "LDS read B")
        got = set()
        for a in range(FR):
            j = j0 + (wr * FR + a) * 16 + 4 * (lane >> 4)
            for b_ in range(FH):
                m = m0 + (wh * FH + b_) * 16 + (lane & 15)
                ok = (m < M) & (j < nn)
                got |= set(zip(m[ok].tolist(), j[ok].tolist()))
                if opos:
                    seq = m // seq_rows if seq_rows else np.zeros_like(m)
                    count = (nseq if seq_rows else batch)
                    base = seq if seq_rows else np.full_like(m, bb)
                    need(np.all(base[ok] < count), "sequence of a hidden row", M, seq_rows, count)
                    ld4 = ok & (j + 3 < opos_len)
                    need(np.all((base * ids_stride + j + 3)[ld4] < count * ids_stride), "column table")
                    need(np.all((opos_len >= nn) | ~ok), "columns of the last rows", opos_len, nn)
                else:
                    vec = ok & (j + 3 < nn)
                    need(np.all((j + 3)[vec] < ld) and np.all(j[ok] < ld), "row end", ld)
        need(got == {(m, j) for m in range(m0, min(m0 + BN, M)) for j in range(j0, min(j0 + BM, nn), 4)}, "every logit of the block once")


def check_shared(rows_total, seq_rows, d, cap_rows, opos_stride, V=128256, nseq=None):
    """launch_head_shared: one id list for all sequences; hidden rows [rows_total][d], column tables [nseq][opos_stride]
    looked up per hidden row at the end.  Beyond 32-bit byte offsets 64 hidden rows at a time."""
    nseq = nseq if nseq is not None else ceil_div(rows_total, seq_rows)
    need(cap_rows >= 64 and cap_rows % 64 == 0 and opos_stride % 4 == 0, "list capacity", cap_rows, opos_stride)
    if choose.wide_reaches(V, rows_total, d):
        for n in (0, 1, cap_rows // 2 + 1, cap_rows):
            check_wide(rows_total, d, V, n, cap_rows, opos_stride, choose.wide_shared_shape(rows_total), ids_stride=opos_stride, opos=True, seq_rows=seq_rows, nseq=nseq)
        return
    groups, tail = rows_total // 64, rows_total % 64
    launches = ([(0, groups, 64)] if groups else []) + ([(groups * 64, 1, tail)] if tail else [])
    for row0, nb, M in launches:
        check_tile64(M, d, nb, cap_rows, 1 << 30, cap_rows, False, MT=2 if M <= 32 else 4, fast=choose.tile64_fast(M, d), split=False, S=ceil_div(d, 512))
        for b in (0, nb - 1):
            for m in range(M):                                 # rows the kernel stores for: m < M
                r = row0 + b * M + m
                need(r < rows_total, "hidden row", r, rows_total)
                q = r // seq_rows
                need(q < nseq, "sequence of a hidden row", q, nseq)
                for j in range(0, cap_rows, 4):
                    if j + 3 < opos_stride:                    # the kernel's own guard
                        need(q * opos_stride + j + 3 < nseq * opos_stride, "column table", q, j)


# ---- head_gemm_kernel -----------------------------------------------------------------------------------------------------
GEMM_WAITS = (10, 8, 8)                                          # fetches that may be in flight at the end of a step's first three clusters


def gemm_events(nk, waits=GEMM_WAITS, prologue_wait=10):
    """One wavefront's program: ("fetch", operand, step, half) -- two instructions each --, ("wait", instructions that may be in flight), ("read", ...),
    ("use",) = the matrix instructions that consume everything read so far, ("bar",)"""
    ev = [("fetch", "a", 0, 0), ("fetch", "b", 0, 0), ("fetch", "b", 0, 1), ("fetch", "a", 0, 1), ("fetch", "a", 1, 0), ("fetch", "b", 1, 0), ("fetch", "b", 1, 1),
          ("wait", prologue_wait), ("bar",), ("read", "b", 0, 0), ("skew",)]
    for st in range(nk):
        ev += [("read", "a", st, 0), ("fetch", "a", st + 1, 1), ("wait", waits[0]), ("bar",), ("use",), ("bar",),
               ("read", "b", st, 1), ("wait", waits[1]), ("bar",), ("use",), ("bar",),
               ("read", "a", st, 1), ("fetch", "a", st + 2, 0), ("fetch", "b", st + 2, 0), ("wait", waits[2]), ("bar",), ("use",), ("bar",),
               ("read", "b", st + 1, 0), ("fetch", "b", st + 2, 1), ("bar",), ("use",), ("bar",)]
    return ev


@functools.lru_cache(maxsize=None)
def check_gemm_schedule(nk, **kw):
    """the second four wavefronts run one barrier behind the first; all eight fetch a share of every piece of LDS and read from all of it"""
    fetched, landed, reads = {}, {}, {}
    bars = []
    for group in (0, 1):
        interval, flight, open_reads = 0, [], []
        for e in gemm_events(nk, **kw):
            if e[0] == "bar" or (e[0] == "skew" and group == 1):
                interval += 1
            elif e[0] == "fetch":
                _, op, st, h = e
                flight += [(op, st, h)] * 2
                fetched[(group, op, st, h)] = interval
            elif e[0] == "wait":
                while len(flight) > e[1]:
                    piece = flight.pop(0)
                    if piece not in flight:
                        landed[(group, *piece)] = interval
            elif e[0] == "read":
                open_reads.append(e[1:])
                reads.setdefault(e[1:], []).append([group, interval, None])
            elif e[0] == "use":
                for r in open_reads:
                    reads[r][-1][2] = interval
                open_reads = []
        bars.append(interval + (1 if group == 0 else 0))          # the first four wavefronts' last barrier
    need(bars[0] == bars[1], "both halves of the workgroup pass the same number of barriers", bars)
    for (op, st, h), rs in reads.items():
        if st >= nk:
            continue                                            # read behind the last step, never used
        for group, at, used in rs:
            for other in (0, 1):
                need(landed.get((other, op, st, h), 1 << 30) < at, "a piece is read before a barrier behind its arrival", op, st, h)
    for (group, op, st, h), at in fetched.items():
        for g2, r_at, used in reads.get((op, st - 2, h), []):    # what the same piece of LDS held before
            need(used is not None and used < at, "a piece is refilled before everybody has used it", op, st, h)


def permuted(piece, row):
    return piece ^ (row & 7)


@functools.lru_cache(maxsize=None)
def check_gemm_operands(nk, d, swizzle):
    """where the fetches put what -- LDS byte -> (row of the block, 16-byte piece of the step) -- and where the fragments are read"""
    lane = LANES
    for op, where in (("a", lambda q, h: (q >> 6) * 128 + (q & 63) + h * 64), ("b", lambda q, h: (q >> 5) * 64 + (q & 31) + h * 32)):
        lds = {}
        for h, w, i in itertools.product((0, 1), range(8), (0, 1)):
            q = (2 * w + i) * 8 + (lane >> 3)
            pc = (lane & 7) ^ (lane >> 3)
            dst = h * 16384 + w * 2048 + i * 1024 + lane * 16
            need(np.all(pc * 16 + (nk - 1) * 128 + 16 <= d * 2), "column bytes")
            for a, r, p in zip(dst.tolist(), where(q, h).tolist(), pc.tolist()):
                need(a not in lds and a + 16 <= 32768, "LDS piece written twice")
                lds[a] = (r, p)
        need(len(lds) == 2048, "the whole operand block")
        for h, wv in itertools.product((0, 1), range(2 if op == "a" else 4)):
            for f, kk in itertools.product(range(4 if op == "a" else 2), (0, 1)):
                fr = lane & 15
                at = h * 16384 + wv * (8192 if op == "a" else 4096) + f * 2048 + fr * 128 + swizzle((lane >> 4) + 4 * kk, lane) * 16
                row = wv * (128 if op == "a" else 64) + (h * (4 if op == "a" else 2) + f) * 16 + fr
                for a, r, p in zip(at.tolist(), row.tolist(), ((lane >> 4) + 4 * kk).tolist()):
                    need(lds.get(a) == (r, p), "a fragment is read where its row and columns were put", op, h, wv, f, kk)


def check_gemm(M, d, V, n, cap_rows, ld, ids_stride=None, opos=False, swizzle=permuted):
    need(d % 64 == 0 and choose.wide_reaches(V, M, d), "whole steps, 32-bit byte offsets")
    check_gemm_schedule(d // 64)
    check_gemm_operands(d // 64, d, swizzle)
    row_blocks, hid_blocks = ceil_div(cap_rows, 256), ceil_div(M, 256)
    blk = np.arange(ceil_div(row_blocks, 8) * hid_blocks * 8)
    hb, rb = (blk >> 3) % hid_blocks, (blk >> 3) // hid_blocks * 8 + (blk & 7)
    live = (rb < row_blocks) & (rb * 256 < n)
    need(len(set(zip(rb[live].tolist(), hb[live].tolist()))) == int(live.sum()) == ceil_div(n, 256) * hid_blocks, "every live block once")
    lane = LANES
    ids_stride = cap_rows if ids_stride is None else ids_stride
    for rb_, hb_ in {(r, h) for r in {0, (n - 1) // 256} for h in (0, hid_blocks - 1) if n}:
        j = rb_ * 256 + np.arange(256)
        j = np.where(j < n, j, rb_ * 256)
        need(np.all(j < ids_stride), "ids")
        m = np.minimum(hb_ * 256 + np.arange(256), M - 1)
        need(np.all(m < M), "H row")
        for a, wr in itertools.product(range(8), range(2)):
            jj = rb_ * 256 + wr * 128 + a * 16 + 4 * (lane >> 4)
            ok = jj < n
            if opos:
                need(np.all((jj + 3 < ids_stride) | ~(ok & (jj + 3 < cap_rows // 4 * 4))) and cap_rows // 4 * 4 >= n, "column table")
            else:
                need(np.all((jj + 3 < ld) | ~(jj + 3 < n)) and n <= ld, "row end")


# ---- the selection's loads ---------------------------------------------------------------------------------------------------
def check_shifted_loads(ld, addr, cbase, EPT=16, take=lambda sh, e: e + sh):
    """topk_select on rows at any 4-byte address: 16-byte loads from the aligned address below a lane's run; element indexes are relative to the row"""
    sh = (addr & 15) >> 2
    p0 = cbase + np.arange(1024) * EPT
    loaded = np.full((1024, EPT + 4), -1)
    for e in range(0, EPT + 4, 4):
        q = p0 - sh + e
        whole = (q >= 0) & (q + 3 < ld)
        need(np.all((addr + 4 * q[whole]) % 16 == 0), "aligned", addr)
        for i in range(4):
            ok = whole | ((q + 3 >= 0) & (q < ld) & (q + i >= 0) & (q + i < ld))
            need(np.all((q + i)[ok] >= 0) and np.all((q + i)[ok] < ld), "row bounds")
            loaded[ok, e + i] = (q + i)[ok]
    v = np.stack([loaded[:, take(sh, e)] for e in range(EPT)], axis=1)
    want = p0[:, None] + np.arange(EPT)
    need(np.all(v == np.where(want < ld, want, -1)), "a lane's run")


def check_stream(ld, n, addr, NW, piece_clamp=True):
    """topk_stream: the row's whole 16-byte pieces in steps, two ahead, and the elements outside them one by one"""
    NT = 64 * NW
    QP = 4 * NT
    head = ((16 - (addr & 15)) & 15) >> 2
    qcap = (ld - head) >> 2
    nq = (n - head) >> 2 if n > head else 0
    steps = ceil_div(nq, QP) if nq > QP else 1
    need(qcap >= 1 and (addr + 4 * head) % 16 == 0, "a whole aligned piece")
    seen = np.zeros(n, int)
    for p in range(ceil_div(steps, 3) * 3 + 2):                  # three steps a turn, loads two ahead
        q = p * QP + np.arange(QP)
        at = np.minimum(q, qcap - 1) if piece_clamp else q
        need(np.all(head + 4 * at + 3 < ld), "piece past the row", p)
        if p < steps:
            live = q[q < nq]
            for e in range(4):
                seen[head + 4 * live + e] += 1
    for tid in range(8):
        x = (tid if tid < head else n) if tid < 4 else head + 4 * nq + tid - 4
        if x < n and x < ld:
            seen[x] += 1
    need(np.all(seen == 1), "every element once", ld, n, addr)


def check(M, d, batch, cap, V, n, dense, aligned=True, opos=False):
    for kernel, prm, m0, mm in plan(V, M, d, batch, cap, dense, aligned=aligned):
        if kernel == "wide":
            ns = n
            if batch > 1:                                        # ragged: full, empty, one row, as given
                ns = [n if b % 4 == 3 else (cap, 0, 1)[b % 4] for b in range(batch)]
            check_wide(mm, d, V, ns, cap, V if dense else cap, batch=batch, dense=dense, opos=opos, **prm)
        elif kernel == "gemm":
            check_gemm(mm, d, V, n, cap, V if dense else cap, opos=opos)
        elif kernel == "quad":
            check_quad(mm, d, batch, cap, V, n, dense, **prm)
        elif kernel == "private":
            check_private(mm, d, batch, cap, V, n, dense, **prm)
        elif kernel == "tile64":
            check_tile64(mm, d, batch, cap, V, n, dense, **prm)


# ---- tests ----------------------------------------------------------------------------------------------------------------
CAPS = [64, 1472, 3776, 4352, 9216, 32064]


@pytest.mark.parametrize("d", [8, 64, 512, 520, 1024, 1032, 1536, 2048, 2056, 3584, 3592, 4096, 4104, 5120, 6144, 8192, 8200])
def test_every_selected_variant_stays_inside_its_buffers_sparse(d):
    for M, batch, cap in itertools.product((1, 4, 5, 8, 9, 13, 16, 17, 31, 32, 33, 63, 64, 70, 300), (1, 2, 9), CAPS):
        for n in (0, cap // 2 + 1, cap) if batch == 1 else (cap // 2 + 1,):
            check(M, d, batch, cap, 128256, n, dense=False)
    for M, cap in itertools.product((1, 8, 16, 17, 32, 64, 100), (64, 1472, 4352)):
        check(M, d, 64, cap, 128256, cap // 2 + 1, dense=False)


@pytest.mark.parametrize("V", [16384, 24001, 50001, 128256, 152064])
def test_every_selected_variant_stays_inside_its_buffers_dense(V):
    for M, d in itertools.product((1, 4, 5, 8, 12, 16, 17, 32, 40, 64, 65, 128, 129, 257, 512), (64, 512, 520, 1536, 3584, 4096, 8192)):
        check(M, d, 1, V, V, V, dense=True)
        if M > 128:
            check(M, d, 1, V, V, V, dense=True, aligned=False)


@pytest.mark.parametrize("cap", [16448, 24576, 49152, 98304, 128256])
def test_many_hidden_rows_on_long_lists_stay_inside_their_buffers(cap):
    for M, d in itertools.product((65, 100, 128, 129, 257, 300, 512), (64, 520, 4096)):
        for n in (0, 1, 257, cap - 1, cap):
            check(M, d, 1, cap, 128256, n, dense=False)
        check(M, d, 1, cap, cap, cap // 2 + 1, dense=False, opos=True)      # the packed buffer: rows in slots, columns per slot


def test_every_block_shape_and_step_count_is_modelled():
    for shape in range(choose.GEMM):
        b = choose.block(shape)
        for d in (8, 64, 72, 128, 136, 256, 384, 512, 640, 1088, 4104):
            for n in (1, 15, 16, 17, 255, 256, 257, 700):
                check_wide(b.WH * b.FH * 16 + 3, d, 50000, n, 704, 704, shape)
    with open(os.path.join(choose.ROOT, "paper_2605_26444_amd", "csrc", "wide.hip")) as f:
        src = f.read()
    src = src[src.index("  // prologue\n"):src.index("  int st = 0;\n")]
    assert [int(x) for x in re.findall(r"NS_WAIT_VM\((\d+)\)", src)] == [10, *GEMM_WAITS]      # the kernel's own counts
    for nk in range(1, 9):
        check_gemm_schedule(nk)
    for M, d, n in ((129, 64, 1), (256, 128, 255), (257, 192, 256), (512, 4096, 257), (1024, 64, 512)):
        check_gemm(M, d, 50000, n, 512, 512)


def test_each_die_takes_its_eighth_of_every_list_once():
    rng = np.random.default_rng(0)
    for shape, batch in itertools.product((0, 1), (8, 9, 33, 64)):
        for cap in (64, 1472, 4096):
            check_wide(8, 72, 50000, rng.integers(0, cap + 1, batch), cap, cap, shape, batch=batch, by_die=True)
            check_wide(8, 72, 50000, [min(cap, b) for b in range(batch)], cap, cap, shape, batch=batch, by_die=True)


def test_shared_list_launches_stay_inside_their_buffers():
    for nseq, seq_rows, d, cap_rows in itertools.product((1, 3, 6, 20, 30, 64), (1, 3, 5, 8, 16, 40), (64, 512, 1032, 4096), (64, 1472)):
        check_shared(nseq * seq_rows, seq_rows, d, cap_rows, cap_rows)
    for rows, d in ((40, 4096), (200, 1032)):                              # a matrix beyond 32-bit byte offsets: 64 hidden rows at a time
        check_shared(rows, 8, d, 1472, 1472, V=4000000)
        check_shared(rows, 8, d, 1472, 64, V=4000000)                      # a column table narrower than the list
    for V in (128256, 4000000):
        with pytest.raises(OutOfBounds):                                   # hidden rows counted per launch, not over the whole batch
            check_shared(160, 8, 4096, 64, 64, V=V, nseq=19)
        with pytest.raises(OutOfBounds):
            check_shared(160, 8, 4096, 96, 96, V=V)


def test_selection_loads_stay_inside_their_rows():
    for ld, off in itertools.product((16385, 16386, 16387, 30001, 32771), (0, 4, 8, 12)):
        for cbase in (0, 16384):
            check_shifted_loads(ld, off, cbase)
        for n in sorted({0, 1, 2, 3, 4, 5, 16384, 16385, ld - 3, ld - 1, ld}):
            for NW in (8, 16):
                check_stream(ld, n, off, NW)
    with pytest.raises(OutOfBounds):
        check_shifted_loads(30001, 8, 0, take=lambda sh, e: e)             # unshifted
    with pytest.raises(OutOfBounds):
        check_stream(30001, 30001, 4, 16, piece_clamp=False)               # two steps ahead without the clamp


def test_the_selection_that_once_faulted_is_rejected():
    """constant hidden-row strides (the M == 64 form) taken with M = 32 and two sequences: the last sequence's
    wavefronts 2-3 would address hidden rows 32..63, past the end of H."""
    with pytest.raises(OutOfBounds):
        check_tile64(32, 8192, 2, 128, 20000, 70, False, MT=2, fast=2, split=True, S=16)
    check_tile64(32, 8192, 2, 128, 20000, 70, False, MT=2, fast=1, split=True, S=16)      # the clamped form is fine
    assert plan(20000, 32, 8192, 2, 128, False)[0][1]["fast"] == 1                        # and is what the launcher takes
    assert plan(20000, 64, 8192, 2, 128, False)[0][1]["fast"] == 2


def test_the_model_rejects_other_planted_mistakes():
    with pytest.raises(OutOfBounds):       # a K-loop kernel's FAST form on a hidden size that is not a whole K-iteration
        check_private(16, 8200, 1, 1472, 128256, 1000, False, RT=1, MT=4, KS=4, NW=4, fast=True)
    with pytest.raises(OutOfBounds):       # two loads per wavefront for more columns than they cover
        check_quad(8, 1032, 1, 1472, 128256, 1000, False, NRG=1, RT=1, MT=2, KS=2)
    with pytest.raises(OutOfBounds):       # whole-slice loads on d % 512 != 0
        check_tile64(64, 3592, 1, 4352, 152064, 3000, False, MT=4, fast=2, split=True, S=8)
    with pytest.raises(OutOfBounds):       # an id list whose capacity is not a whole number of row groups
        check_private(8, 8192, 1, 1470, 128256, 1000, False, RT=2, MT=2, KS=8, NW=4, fast=True)
    with pytest.raises(OutOfBounds):       # split-K planes larger than the workspace
        check_tile64(64, 3584, 1, 4352, 152064, 3000, False, MT=4, fast=2, split=True, S=7, partial_elems=1000)
    shape = choose.wide_shape(64, 4096, 1, 4352)
    with pytest.raises(OutOfBounds):       # the form without a tail on a hidden size that is not a whole number of steps
        check_wide(64, 3592, 152064, 3000, 4352, 4352, shape, tail=False)
    with pytest.raises(OutOfBounds):       # logits rows shorter than the row count
        check_wide(64, 4096, 20000, 4352, 4352, 4348, shape)
    with pytest.raises(OutOfBounds):       # an odd number of register sets
        check_wide(64, 4096, 20000, 3000, 4352, 4352, shape, blocks=choose.block(shape)._replace(D=3))
    with pytest.raises(OutOfBounds):       # rows beyond the reach of the byte offsets
        check_wide(64, 8192, 300000, 3000, 4352, 4352, shape)
    with pytest.raises(OutOfBounds):       # the pieces of a fragment read without their permutation
        check_gemm(512, 4096, 50000, 700, 704, 704, swizzle=lambda piece, row: piece)
    for waits in ((12, 8, 8), (10, 10, 8), (10, 8, 10)):       # one fetch too many may be in flight
        with pytest.raises(OutOfBounds):
            check_gemm_schedule(6, waits=waits)
    with pytest.raises(OutOfBounds):
        check_gemm_schedule(6, prologue_wait=12)
