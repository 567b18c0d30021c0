"""The launchers' own choice of kernel and block shape (csrc/choose.h, plain host arithmetic), compiled with g++ for the CPU
tests.  Not collected by pytest."""
from __future__ import annotations

import ctypes as C
import os
import subprocess
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_ABI = r"""
#include "choose.h"
using namespace nanospec;
extern "C" {
int c_wide_supported(int V, int M, int d, int batch, int cap, int dense) { return wide_supported(V, M, d, batch, cap, dense != 0); }
int c_wide_reaches(int V, int M, int d) { return wide_reaches(V, M, d); }
int c_wide_shape(int M, int d, int batch, int cap, int dense, int aligned) { return wide_shape(M, d, batch, cap, dense != 0, aligned != 0); }
int c_wide_by_die(int M, int batch, int cap, int dense) { return wide_by_die(M, batch, cap, dense != 0); }
int c_wide_shared_shape(int rows) { return wide_shared_shape(rows); }
void c_wide_block(int shape, int* o) { const WideBlock b = kWideBlocks[shape]; o[0] = b.WR; o[1] = b.WH; o[2] = b.FR; o[3] = b.FH; o[4] = b.BK; o[5] = b.D; }
int c_gemm_shape() { return kWideGemm; }
void c_quad_plan(int M, int d, int batch, int cap, int dense, int* o) {
  const QuadPlan q = quad_plan(M, d, batch, cap, dense != 0);
  o[0] = q.MT; o[1] = q.KS; o[2] = q.NRG; o[3] = q.RT; o[4] = q.loop;
}
int c_head_split(int M, int d, int batch, int cap, int dense, long long partial_bytes, long long ld) { return head_split(M, d, batch, cap, dense != 0, partial_bytes, ld); }
int c_vocab_init_serial(int batch, int window, int longest) { return vocab_init_serial(batch, window, longest); }
int c_topk_chunks(int list, long long rows, int k, int topk_cap, int window, int distinct) { return topk_chunks(list != 0, rows, k, topk_expected(topk_cap, window, distinct != 0)); }
int c_hold_supported(int V, int M, int d, int batch, int cap, int dense) { return hold_supported(V, M, d, batch, cap, dense != 0); }
void c_hold_plan(int d, int batch, int dense, int M, int* o) {
  const HoldPlan h = hold_plan(d, batch, dense != 0);
  o[0] = h.NW; o[1] = h.parts; o[2] = h.seg; o[3] = (int)hold_lds(h, M);
}
int c_kslice_supported(int V, int M, int d, int batch, int cap, int dense, int aligned) { return kslice_supported(V, M, d, batch, cap, dense != 0, aligned != 0); }
void c_kslice_plan(int M, int batch, int cap, int* o) {
  const SlicePlan p = kslice_plan(M, batch, cap);
  o[0] = p.LB; o[1] = p.parts; o[2] = p.hid_blocks; o[3] = p.rows;
}
int c_union_feeds(int batch, int cap) { return union_feeds(batch, cap); }
int c_union_split_pairs(int pairs, int rest) { return union_split_pairs(pairs, rest); }
int c_union_split(int M, int d, int batch, int cap) { return union_split(M, d, batch, cap); }
int c_tile64_fast(int M, int d) { return tile64_fast(M, d); }
}
"""

Quad = namedtuple("Quad", "MT KS NRG RT loop")
Block = namedtuple("Block", "WR WH FR FH BK D")
Slice = namedtuple("Slice", "LB parts hid_blocks rows")
Hold = namedtuple("Hold", "NW parts seg lds")


def _load():
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "choose.cpp"), os.path.join(tmp, "choose.so")
        with open(src, "w") as f:
            f.write(_ABI)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2605_26444_amd", "csrc"), "-o", so, src],
                       check=True)
        return C.CDLL(so)


_lib = _load()
_lib.c_head_split.argtypes = [C.c_int] * 5 + [C.c_longlong] * 2
_lib.c_topk_chunks.argtypes = [C.c_int, C.c_longlong] + [C.c_int] * 4
GEMM = _lib.c_gemm_shape()


def wide_supported(V, M, d, batch, cap, dense=False):
    return bool(_lib.c_wide_supported(V, M, d, batch, cap, int(dense)))


def hold_supported(V, M, d, batch, cap, dense=False):
    return bool(_lib.c_hold_supported(V, M, d, batch, cap, int(dense)))


def hold_plan(d, batch, M, dense=False):
    o = (C.c_int * 4)()
    _lib.c_hold_plan(d, batch, int(dense), M, o)
    return Hold(*o)


def kslice_supported(V, M, d, batch, cap, dense=False, aligned=True):
    return bool(_lib.c_kslice_supported(V, M, d, batch, cap, int(dense), int(aligned)))


def kslice_plan(M, batch, cap):
    o = (C.c_int * 4)()
    _lib.c_kslice_plan(M, batch, cap, o)
    return Slice(*o)


def union_split(M, d, batch, cap):
    return bool(_lib.c_union_split(M, d, batch, cap))


def union_feeds(batch, cap):
    return bool(_lib.c_union_feeds(batch, cap))


def union_split_pairs(pairs, rest):
    return bool(_lib.c_union_split_pairs(pairs, rest))


def wide_reaches(V, M, d):
    return bool(_lib.c_wide_reaches(V, M, d))


def wide_shape(M, d, batch, cap, dense=False, aligned=True):
    return _lib.c_wide_shape(M, d, batch, cap, int(dense), int(aligned))


def wide_by_die(M, batch, cap, dense=False):
    return bool(_lib.c_wide_by_die(M, batch, cap, int(dense)))


def wide_shared_shape(rows_total):
    return _lib.c_wide_shared_shape(rows_total)


def block(shape):
    o = (C.c_int * 6)()
    _lib.c_wide_block(shape, o)
    return Block(*o)


def rows_by_hidden(shape):
    """'64x32': logit rows x hidden rows of a block"""
    b = block(shape)
    return "gemm" if shape == GEMM else f"{b.WR * b.FR * 16}x{b.WH * b.FH * 16}"


def quad_plan(M, d, batch, cap, dense=False):
    o = (C.c_int * 5)()
    _lib.c_quad_plan(M, d, batch, cap, int(dense), o)
    return Quad(*o[:4], bool(o[4]))


def head_split(M, d, batch, cap, dense, partial_bytes, ld):
    return bool(_lib.c_head_split(M, d, batch, cap, int(dense), partial_bytes, ld))


def tile64_fast(M, d):
    return _lib.c_tile64_fast(M, d)


def vocab_init_serial(batch, window, longest):
    return bool(_lib.c_vocab_init_serial(batch, window, longest))


def topk_chunks(rows, k, topk_cap=0, window=0, distinct=False, dense=False):
    return bool(_lib.c_topk_chunks(int(not dense), rows, k, topk_cap, window, int(distinct)))
