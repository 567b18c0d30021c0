"""Selection on rows longer than one workgroup's registers: one workgroup per row in steps, for lists and for many dense
rows, and the chunks of few dense rows.  Row strides of every alignment, counts around the step and piece boundaries, and
the inputs that overflow the candidate list: ramps, plateaus, all values equal.  Ids and values must be exactly those of a
stable descending sort (ties by lower id); log-probabilities within 1e-5 of the fp64 value (an fp32 sum of at most 1e5 positive
terms per row, added in trees of 4 and 6 levels behind runs of 16: below 2e-6 relative)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_26444_amd import binding as B

from harness import csr, dev_ids

pytestmark = pytest.mark.gpu


def _rows(kind, rows, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + rows)
    x = torch.empty((rows, n), device="cuda").normal_(generator=g)
    i = torch.arange(n, device="cuda", dtype=torch.float32)
    if kind == "up":
        return (i * 1e-3).expand(rows, n).contiguous()
    if kind == "down":
        return (-i * 1e-3).expand(rows, n).contiguous()
    if kind == "equal":
        return torch.zeros((rows, n), device="cuda")
    if kind == "plateaus":
        return torch.floor(i / 5000).expand(rows, n).contiguous()
    if kind == "coarse":
        return torch.round(x * 2) / 2
    return x


def _expect(x, k):
    v, i = torch.sort(x, dim=1, descending=True, stable=True)
    k2 = min(k, x.shape[1])
    return i[:, :k2], v[:, :k2]


@pytest.mark.parametrize("kind", ["normal", "up", "down", "equal", "plateaus", "coarse"])
@pytest.mark.parametrize("rows,V,k", [(1, 16385, 64), (3, 40003, 10), (95, 16386, 1), (96, 32771, 40), (130, 50001, 64), (512, 16387, 3), (515, 24589, 64)])
def test_dense_rows(kind, rows, V, k):
    x = _rows(kind, rows, V)
    nbytes = B.nanospec_dense_topk_workspace(V, rows, k)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    ids = torch.full((rows, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((rows, k), 9.0, device="cuda")
    B.nanospec_dense_topk(x, V, rows, k, ids, vals, ws, nbytes)
    ei, ev = _expect(x, k)
    assert torch.equal(ids.long(), ei) and torch.equal(vals, ev)


@pytest.mark.parametrize("kind", ["normal", "up", "equal", "coarse"])
@pytest.mark.parametrize("n", [0, 1, 37, 8191, 8192, 8193, 16384, 16385, 16388, 32768, 32770, 39999])
@pytest.mark.parametrize("batch,M,k", [(2, 3, 10), (1, 2, 64), (16, 32, 5)])
@pytest.mark.parametrize("room", ["window", "candidates"])
def test_lists(kind, n, batch, M, k, room):
    """one workgroup per row, and -- room for a candidate set of the list's length -- chunks"""
    V, window, T = 60000, 40000, 1
    if room == "candidates":
        V, window, T = 90000, 1000, 39999 if k <= 16 else 70000
    st = B.State(V, 8, batch, window, T, M, k)
    assert st.capacity > 16384
    rng = np.random.default_rng(n + 1)
    live = [n if b % 2 == 0 else n // 3 for b in range(batch)]
    lists = [np.sort(rng.permutation(V)[:x]).astype(np.int32) for x in live]
    flat, off = csr(lists)
    none = np.zeros(batch + 1, np.int32)
    if room == "window":
        B.nanospec_vocab_init(st.h, dev_ids(flat), off, None, none)
    else:
        B.nanospec_vocab_init(st.h, None, none, dev_ids(flat), off)
    logits = torch.full((batch, M, st.capacity), 1e30, device="cuda")       # what lies behind a list must not matter
    ids = torch.full((batch, M, k), -7, dtype=torch.int32, device="cuda")
    vals, logp = torch.full((batch, M, k), 9.0, device="cuda"), torch.full((batch, M, k), 9.0, device="cuda")
    for b in range(batch):
        if live[b]:
            logits[b, :, :live[b]] = _rows(kind, M, live[b])
    B.nanospec_topk_remap(st.h, logits, M, k, ids, vals)
    ids2 = torch.full_like(ids, -7)
    B.nanospec_topk_logprob_remap(st.h, logits, M, k, ids2, logp)
    assert torch.equal(ids, ids2)
    for b in range(batch):
        have = min(k, live[b])
        assert torch.all(ids[b, :, have:] == -1) and torch.all(vals[b, :, have:] == -torch.inf) and torch.all(logp[b, :, have:] == -torch.inf)
        if have:
            x = logits[b, :, :live[b]]
            ei, ev = _expect(x, k)
            assert torch.equal(ids[b, :, :have].long(), torch.from_numpy(lists[b]).long().cuda()[ei]) and torch.equal(vals[b, :, :have], ev)
            z = ev.double() - torch.logsumexp(x.double(), dim=1, keepdim=True)
            assert torch.all((logp[b, :, :have].double() - z).abs() <= 1e-5 * (1 + z.abs())), b
    st.close()


def _without(x, how, what=torch.nan):
    """`what` in the first piece or nearly everywhere, or at single places at the row's ends and across the pieces"""
    n = x.shape[1]
    x = x.clone()
    if how == "all":
        x[:] = what
    elif how == "front":
        x[:, :min(n, 16400)] = what
    elif how == "front_but_few":
        keep = x[:, 100:120].clone()
        x[:, :min(n, 16400)] = what
        x[:, 100:120] = keep
    elif how == "all_but_few":
        keep = x[:, n // 2:n // 2 + 7].clone()
        x[:] = what
        x[:, n // 2:n // 2 + 7] = keep
    else:
        x[:, ::3] = what
        x[:, :3] = what
        x[:, -3:] = what
    return x


def _check_missing(x, ids, vals, k, names=None):
    """x: logits with -inf where an element cannot be selected; slots without one hold -1 and -inf"""
    ei, ev = _expect(x, k)
    none = ev == -torch.inf
    ei = ei if names is None else names[ei]
    assert torch.equal(ids.long(), torch.where(none, -1, ei)) and torch.equal(vals, ev)


HOW = ["all", "front", "front_but_few", "all_but_few", "scattered"]


@pytest.mark.parametrize("how", HOW)
@pytest.mark.parametrize("rows,V,k", [(96, 32771, 40), (515, 24589, 64)])
def test_dense_rows_with_nans(how, rows, V, k):
    """rows walked by one workgroup: NaN logits are no candidates, a row has fewer winners and the slots left over are padding"""
    x = _without(_rows("normal", rows, V), how)
    nbytes = B.nanospec_dense_topk_workspace(V, rows, k)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    ids = torch.full((rows, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((rows, k), 9.0, device="cuda")
    B.nanospec_dense_topk(x, V, rows, k, ids, vals, ws, nbytes)
    _check_missing(torch.nan_to_num(x, nan=-torch.inf), ids, vals, k)


@pytest.mark.parametrize("how", HOW)
@pytest.mark.parametrize("n", [16388, 32770, 39999])
@pytest.mark.parametrize("batch,M,k", [(2, 3, 10), (1, 2, 64), (16, 32, 5)])
def test_lists_with_nans(how, n, batch, M, k):
    V, window = 60000, 40000
    st = B.State(V, 8, batch, window, 1, M, k)
    ids_of = np.sort(np.random.default_rng(n).permutation(V)[:n]).astype(np.int32)
    flat, off = csr([ids_of] * batch)
    B.nanospec_vocab_init(st.h, dev_ids(flat), off, None, np.zeros(batch + 1, np.int32))
    logits = torch.full((batch, M, st.capacity), 1e30, device="cuda")
    x = _without(_rows("normal", batch * M, n), how)
    logits[:, :, :n] = x.view(batch, M, n)
    ids, vals = torch.full((batch * M, k), -7, dtype=torch.int32, device="cuda"), torch.full((batch * M, k), 9.0, device="cuda")
    B.nanospec_topk_remap(st.h, logits, M, k, ids, vals)
    ids2, logp = torch.full_like(ids, -7), torch.empty_like(vals)
    B.nanospec_topk_logprob_remap(st.h, logits, M, k, ids2, logp)
    _check_missing(torch.nan_to_num(x, nan=-torch.inf), ids, vals, k, torch.from_numpy(ids_of).long().cuda())
    assert torch.equal(ids, ids2)
    st.close()


@pytest.mark.parametrize("how", HOW)
@pytest.mark.parametrize("rows,V,k,T", [(3, 40003, 10, 1), (3, 40003, 10, 20000), (96, 32771, 40, 1), (515, 24589, 64, 1)])
def test_rows_with_minus_infinity(how, rows, V, k, T):
    """in a long row a logit of -inf (a masked token) is an empty slot, as a dense row and as a list of the same length"""
    x = _without(_rows("normal", rows, V), how, -torch.inf)
    nbytes = B.nanospec_dense_topk_workspace(V, rows, k)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    ids = torch.full((rows, k), -7, dtype=torch.int32, device="cuda")
    vals = torch.full((rows, k), 9.0, device="cuda")
    B.nanospec_dense_topk(x, V, rows, k, ids, vals, ws, nbytes)
    _check_missing(x, ids, vals, k)
    st = B.State(V, 8, 1, V, T, rows, k)
    names = torch.arange(V, dtype=torch.int32, device="cuda")
    B.nanospec_vocab_init(st.h, names, np.array([0, V], np.int32), None, np.zeros(2, np.int32))
    logits = torch.full((rows, st.capacity), 1e30, device="cuda")
    logits[:, :V] = x
    ids2, vals2 = torch.full_like(ids, -7), torch.full_like(vals, 9.0)
    B.nanospec_topk_remap(st.h, logits, rows, k, ids2, vals2)
    assert torch.equal(ids, ids2) and torch.equal(vals, vals2)
    B.nanospec_topk_logprob_remap(st.h, logits, rows, k, ids2, vals2)
    assert torch.equal(ids, ids2)
    z = torch.where(vals == -torch.inf, vals.double(), vals.double() - torch.logsumexp(x.double(), dim=1, keepdim=True))
    assert torch.equal(vals2 == -torch.inf, z == -torch.inf)
    assert torch.all(torch.where(z == -torch.inf, 0.0, (vals2.double() - z).abs()) <= 1e-5 * (1 + torch.where(z == -torch.inf, 0.0, z.abs())))
    st.close()
