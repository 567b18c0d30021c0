"""The head with its hidden rows in registers, at the sizes where it can go wrong: hidden sizes that do not fill a wavefront's 1024 columns (down to one
16-byte piece of the last one), pieces of no rows, one row, a last quad of one to three, several segments, empty lists beside full ones, rows kept in an order
of their own.  Against fp64; the bound is that of an fp32 sum of d exact products in any order, d * 2^-24 * sum |w h|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import choose
from paper_2605_26444_amd import binding as B

from harness import csr, dev_ids

pytestmark = pytest.mark.gpu


def _normal(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)


def _check(got, W, H, what):
    w, h = W.double(), H.double()
    bound = W.shape[1] * 2.0 ** -24 * (h.abs() @ w.abs().T)
    assert torch.all((got.double() - h @ w.T).abs() <= bound), what


def _lists(V, batch, M, d, window, sizes, W, H):
    rng = np.random.default_rng(batch * 1000 + M)
    n = np.minimum(np.resize(sizes, batch), window)
    ids = [np.sort(rng.permutation(V)[:x]).astype(np.int32) for x in n]
    st = B.State(V, d, batch, window, 1, M, 1)
    assert choose.hold_supported(V, M, d, batch, st.capacity)
    flat, off = csr(ids)
    B.nanospec_vocab_init(st.h, dev_ids(flat) if len(flat) else None, off, None, np.zeros(batch + 1, np.int32))
    logits = torch.full((batch, M, st.capacity), 7.0, dtype=torch.float32, device="cuda")
    B.nanospec_sparse_head(st.h, W, H, M, logits)
    return st, ids, logits


@pytest.mark.parametrize("batch,M,d,window,sizes", [
    (1, 16, 8192, 9000, [0]), (1, 16, 8192, 9000, [1]), (1, 13, 8192, 9000, [257]), (1, 9, 8184, 9000, [8999]), (1, 5, 5128, 5200, [1100]), (1, 8, 7168, 6000, [5999]),
    (1, 16, 4096, 4300, [4300]), (1, 1, 4096, 4300, [2047]), (1, 4, 2056, 4300, [770]), (1, 8, 3592, 9000, [8195]), (1, 8, 2048, 17000, [16999]), (1, 12, 2048, 33000, [511]),
    (2, 3, 2560, 8200, [6000, 0]), (4, 16, 6144, 2100, [2100, 0, 1, 259]), (7, 5, 4096, 1000, [1000, 3, 0]), (48, 8, 4096, 2100, [500, 17, 64]), (16, 1, 2048, 2100, [999, 8, 0]),
    (64, 8, 2048, 4200, [4200, 2051, 0, 1]), (32, 16, 2568, 2300, [2300, 2049, 2, 257]), (128, 2, 3080, 1100, [200, 9]), (3, 16, 4104, 2600, [2000, 5]), (4, 4, 8192, 2000, [2000, 1999]),
])
def test_lists(batch, M, d, window, sizes):
    V = 20000 if window < 20000 else 34000
    W, H = _normal(1, V, d), _normal(2, batch, M, d)
    st, ids, logits = _lists(V, batch, M, d, window, sizes, W, H)
    for b in range(batch):
        n = len(ids[b])
        if n:
            _check(logits[b, :, :n], W[torch.from_numpy(ids[b]).long().cuda()], H[b], b)
        assert torch.all(logits[b, :, n:] == 7.0), b
    st.close()


@pytest.mark.parametrize("M,d,V", [(9, 4096, 16387), (16, 4096, 131075), (13, 8192, 16384)])
def test_dense(M, d, V):
    assert choose.hold_supported(V, M, d, 1, V, dense=True)
    W, H = _normal(3, V, d), _normal(4, M, d)
    logits = torch.zeros((M, V), dtype=torch.float32, device="cuda")
    B.nanospec_dense_head(W, H, V, d, M, logits)
    for c in range(0, V, 8192):
        _check(logits[:, c:c + 8192], W[c:c + 8192], H, c)


def test_rows_in_an_order_of_their_own():
    V, d, M, window = 20000, 4096, 8, 5200
    W, H = _normal(5, V, d), _normal(6, 1, M, d)
    rng = np.random.default_rng(1)
    st = B.State(V, d, 1, window, 1, M, 1)
    B.nanospec_packed_enable(st.h)
    first = rng.permutation(V)[:window].astype(np.int32)
    B.nanospec_vocab_init(st.h, dev_ids(first), [0, window], None, np.zeros(2, np.int32))
    B.nanospec_packed_gather(st.h, W)
    new = rng.permutation(V)[:900].astype(np.int32)
    B.nanospec_vocab_update(st.h, dev_ids(new), [0, 900], None, None)
    B.nanospec_packed_gather(st.h, W)
    logits = torch.full((1, M, st.capacity), 7.0, dtype=torch.float32, device="cuda")
    assert choose.hold_supported(st.capacity, M, d, 1, st.capacity)
    B.nanospec_packed_head(st.h, H, M, logits)
    act = st.read_active()[0]
    assert np.array_equal(act, np.unique(np.concatenate([first, new])[-window:]))
    _check(logits[0, :, :len(act)], W[torch.from_numpy(act).long().cuda()], H[0], "packed")
    st.close()


def test_infinities_at_a_row_s_start_stay_infinities():
    """columns past d are fetched from the row's start; they must not turn an infinity there into a NaN"""
    V, d, M = 20000, 3592, 8
    W, H = _normal(7, V, d), _normal(8, 1, M, d).abs()
    W[:, 0] = float("inf")
    st, ids, logits = _lists(V, 1, M, d, 6000, [5000], W, H)
    assert torch.all(torch.isposinf(logits[0, :, :5000]))
    st.close()


def off_alignment(t):
    """the same values 8 bytes past a 16-byte boundary"""
    buf = torch.zeros(t.numel() + 4, dtype=t.dtype, device="cuda")
    buf[4:].copy_(t.reshape(-1))
    out = buf[4:].view(t.shape)
    assert out.data_ptr() % 16 == 8
    return out


@pytest.mark.parametrize("batch,M,d,window,sizes", [(1, 16, 8192, 9000, [1500]), (1, 8, 3592, 9000, [8195]), (8, 6, 4096, 2300, [2300, 9])])
def test_operands_off_alignment(batch, M, d, window, sizes):
    V = 20000
    W, H = off_alignment(_normal(9, V, d)), off_alignment(_normal(10, batch, M, d))
    st, ids, logits = _lists(V, batch, M, d, window, sizes, W, H)
    for b in range(batch):
        n = len(ids[b])
        _check(logits[b, :, :n], W[torch.from_numpy(ids[b]).long().cuda()], H[b], b)
        assert torch.all(logits[b, :, n:] == 7.0), b
    st.close()


def check_nan_rows(st, ids, logits, W, H, nan_id, nan_row):
    """a NaN in a listed row or a hidden row stays in that column or row: all other logits are as without it"""
    n = len(ids)
    got, bad = logits[0, :, :n], torch.from_numpy(ids == nan_id).cuda()
    assert bad.sum() == 1 and torch.all(torch.isnan(got[:, bad])) and torch.all(torch.isnan(got[nan_row]))
    rows = [m for m in range(got.shape[0]) if m != nan_row]
    _check(got[rows][:, ~bad], W[torch.from_numpy(ids).long().cuda()][~bad], H[0, rows], "beside NaN")
    st.close()


@pytest.mark.parametrize("M,d", [(8, 3592), (13, 4096)])
def test_nan_stays_in_its_row(M, d):
    V, n = 20000, 4999
    W, H = _normal(11, V, d), _normal(12, 1, M, d)
    nan_id = int(np.sort(np.random.default_rng(1000 + M).permutation(V)[:n])[n - 2])   # beside the copies of the last row
    W[nan_id, d - 1] = float("nan")
    H[0, M - 1, 0] = float("nan")                                                        # the row that stands in for those past M
    st, ids, logits = _lists(V, 1, M, d, 6000, [n], W, H)
    check_nan_rows(st, ids[0], logits, W, H, nan_id, M - 1)
