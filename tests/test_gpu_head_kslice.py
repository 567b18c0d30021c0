"""The head with K sliced over the wavefronts at the sizes where it can go wrong: blocks of every multiple of 8 rows and hidden rows, the last ones partly filled, pieces of no rows and
of several blocks, hidden sizes that end inside a step (down to one 16-byte piece) or leave wavefronts without a step, empty lists beside full ones, rows in an order of their own.
Against fp64; the bound is that of an fp32 sum of d exact products in any order, d * 2^-24 * sum |w h|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import choose
from paper_2605_26444_amd import binding as B

from harness import csr, dev_ids
from test_gpu_head_hold import _check, _normal, check_nan_rows

pytestmark = pytest.mark.gpu


def _run(V, batch, M, d, window, n, W, H):
    rng = np.random.default_rng(batch * 1000 + M)
    ids = [np.sort(rng.permutation(V)[:x]).astype(np.int32) for x in n]
    st = B.State(V, d, batch, window, 1, M, 1)
    assert choose.kslice_supported(V, M, d, batch, st.capacity)
    flat, off = csr(ids)
    B.nanospec_vocab_init(st.h, dev_ids(flat) if len(flat) else None, off, None, np.zeros(batch + 1, np.int32))
    logits = torch.full((batch, M, st.capacity), 7.0, dtype=torch.float32, device="cuda")
    B.nanospec_sparse_head(st.h, W, H, M, logits)
    return st, ids, logits


@pytest.mark.parametrize("M", [17, 24, 25, 32, 33, 40, 41, 48, 49, 56, 64])
@pytest.mark.parametrize("batch,d,window,sizes", [(1, 1024, 2000, (0, 1, 7, 129, 700, 1100, 1150, 1999, 2000)), (1, 2056, 9000, (2500, 5200, 9000)), (3, 1096, 1500, (1500, 0, 3, 801, 1499)), (1, 4040, 640, (640, 365))])
def test_blocks(M, batch, d, window, sizes):
    V = 12000
    W, H = _normal(1, V, d), _normal(2, batch, M, d)
    for first in range(0, len(sizes), batch):
        n = [sizes[(first + b) % len(sizes)] for b in range(batch)]
        st, ids, logits = _run(V, batch, M, d, window, n, W, H)
        for b in range(batch):
            if n[b]:
                _check(logits[b, :, :n[b]], W[torch.from_numpy(ids[b]).long().cuda()], H[b], (b, n))
            assert torch.all(logits[b, :, n[b]:] == 7.0), (b, n)
        st.close()


@pytest.mark.parametrize("batch,M,d,window,sizes", [
    (1, 20, 512, 3000, [2999]), (1, 64, 520, 2900, [1500]), (1, 64, 8192, 20400, [20399]), (1, 17, 4096, 24500, [24100]), (16, 20, 4096, 1700, [1700, 17, 0]), (8, 60, 2048, 2000, [2000, 1, 1800]), (13, 33, 3000, 2000, [2000, 64]),
])
def test_sizes_of_its_range(batch, M, d, window, sizes):
    V = 70000 if window > 16000 else 20000
    W, H = _normal(3, V, d), _normal(4, batch, M, d)
    n = [sizes[b % len(sizes)] for b in range(batch)]
    st, ids, logits = _run(V, batch, M, d, window, n, W, H)
    for b in range(batch):
        if n[b]:
            _check(logits[b, :, :n[b]], W[torch.from_numpy(ids[b]).long().cuda()], H[b], b)
        assert torch.all(logits[b, :, n[b]:] == 7.0), b
    st.close()


def test_rows_in_an_order_of_their_own_and_operands_off_alignment():
    V, d, M, window = 20000, 1032, 40, 3000
    W, H = _normal(7, V, d), _normal(8, 1, M, d)
    rng = np.random.default_rng(1)
    st = B.State(V, d, 1, window, 1, M, 1)
    B.nanospec_packed_enable(st.h)
    first, new = rng.permutation(V)[:window].astype(np.int32), rng.permutation(V)[:700].astype(np.int32)
    B.nanospec_vocab_init(st.h, dev_ids(first), [0, window], None, np.zeros(2, np.int32))
    B.nanospec_packed_gather(st.h, W)
    B.nanospec_vocab_update(st.h, dev_ids(new), [0, 700], None, None)
    B.nanospec_packed_gather(st.h, W)
    logits = torch.full((1, M, st.capacity), 7.0, dtype=torch.float32, device="cuda")
    assert choose.kslice_supported(st.capacity, M, d, 1, st.capacity)
    B.nanospec_packed_head(st.h, H, M, logits)
    act = st.read_active()[0]
    rows = W[torch.from_numpy(act).long().cuda()]
    _check(logits[0, :, :len(act)], rows, H[0], "packed")
    odd = torch.zeros(M * d + 4, dtype=torch.bfloat16, device="cuda")          # hidden rows 8 bytes off: no fetches into LDS
    odd[4:].copy_(H.reshape(-1))
    logits.fill_(7.0)
    B.nanospec_sparse_head(st.h, W, odd[4:].reshape(1, M, d), M, logits)
    _check(logits[0, :, :len(act)], rows, H[0], "8 bytes off")
    st.close()


def test_infinities_at_a_row_s_start_stay_infinities():
    """columns past d are fetched from the row's start; they must not turn an infinity there into a NaN"""
    V, d, M, n = 9000, 1032, 20, 1500
    W, H = _normal(9, V, d), _normal(10, 1, M, d).abs()
    W[:, 0] = float("inf")
    st, ids, logits = _run(V, 1, M, d, 2000, [n], W, H)
    assert torch.all(torch.isposinf(logits[0, :, :n]))
    st.close()


def test_nan_stays_in_its_row():
    """also where the last fragment's second half is whatever lies behind it in LDS"""
    V, d, M, n = 9000, 1032, 20, 1499
    W, H = _normal(11, V, d), _normal(12, 1, M, d)
    nan_id = int(np.sort(np.random.default_rng(1000 + M).permutation(V)[:n])[n - 2])
    W[nan_id, d - 1] = float("nan")
    H[0, M - 1, 0] = float("nan")
    st, ids, logits = _run(V, 1, M, d, 2000, [n], W, H)
    check_nan_rows(st, ids[0], logits, W, H, nan_id, M - 1)
