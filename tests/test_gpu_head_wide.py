"""The register-blocked head on every block shape it is launched in: ragged batches with an
empty and a one-row list, lists that end inside a block, hidden sizes that are no whole number of column steps (down to
one 16-byte piece) or an odd number of them, hidden rows that end inside a block.  Against fp64; the bound is that of an
fp32 sum of d exact products in any order, d * 2^-24 * sum |w h|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

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


@pytest.mark.parametrize("batch,M,d,window", [
    (1, 17, 8, 100), (1, 64, 520, 3000), (2, 33, 640, 700), (4, 32, 1096, 3000),       # 32 x 32
    (2, 70, 264, 300),                                                                 # ... more hidden rows than 64 per sequence
    (1, 64, 4104, 2500), (1, 20, 2056, 700),                                           # both sides of the split-K line
    (3, 64, 136, 4100), (3, 40, 384, 4100),                                            # 32 x 64
    (7, 64, 200, 4100), (5, 50, 768, 5000),                                            # 64 x 64
    (40, 20, 72, 2000), (40, 32, 264, 2000),                                           # 64 x 32
    (30, 64, 72, 4000), (30, 35, 192, 4000),                                           # 128 x 64
    (1, 16, 520, 9200), (3, 9, 4168, 3100), (1, 3, 1032, 8200), (9, 8, 72, 4100),      # 32 x 16
    (16, 8, 2056, 4700), (8, 16, 200, 4100), (11, 9, 72, 1100),                        # ... each die its eighth of the lists
    (33, 1, 200, 4100), (33, 16, 640, 4100), (33, 7, 4104, 4100),                      # 64 x 16
    (1, 16, 520, 16400), (1, 9, 4096, 9200), (1, 3, 1032, 24600), (1, 7, 2056, 12300), (3, 9, 4168, 5500),   # 32 x 16, on either side of its lines
    (1, 16, 520, 16300), (1, 9, 4096, 9100), (1, 3, 1032, 24500), (1, 7, 2056, 12200), (3, 9, 4168, 5400),
    (9, 8, 72, 7400), (9, 1, 4096, 7400), (11, 9, 72, 1900), (9, 8, 72, 7200), (11, 9, 72, 1800),            # ... each die its eighth
    (2, 17, 4104, 2500), (2, 64, 3080, 2000), (2, 64, 3080, 2100), (8, 33, 4096, 300), (2, 17, 8192, 9200), (2, 20, 2048, 1000), (2, 20, 12288, 2500),   # split-K and beside it
    (4, 3, 264, 33000), (4, 8, 5128, 33000),                                                                 # 64 x 16, and not beyond d = 5120
])
def test_ragged_batches(batch, M, d, window):
    V = 20000 if window < 20000 else 34000
    rng = np.random.default_rng(batch * 1000 + M)
    n = rng.integers(window // 2, window + 1, batch)
    n[0] = window
    if batch > 2:
        n[1], n[2] = 0, 1
    ids = [np.sort(rng.permutation(V)[:x]).astype(np.int32) for x in n]
    W, H = _normal(1, V, d), _normal(2, batch, M, d)
    st = B.State(V, d, batch, window, 1, M, 1)
    flat, off = csr(ids)
    B.nanospec_vocab_init(st.h, dev_ids(flat), off, None, np.zeros(batch + 1, np.int32))
    logits = torch.full((batch, M, st.capacity), 7.0, dtype=torch.float32, device="cuda")
    B.nanospec_sparse_head(st.h, W, H, M, logits)
    for b in range(batch):
        _check(logits[b, :, :n[b]], W[torch.from_numpy(ids[b]).long().cuda()], H[b], b)
    st.close()


@pytest.mark.parametrize("M", [1, 4, 5, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("d", [8, 520, 1024, 1032, 1536, 2048, 2056])
def test_few_hidden_rows_short_rows(M, d):
    """the kernels that feed the matrix cores from memory, around the hidden sizes where their number of loads changes"""
    for batch, window in ((1, 300), (2, 1100), (4, 2500)):
        test_ragged_batches(batch, M, d, window)


@pytest.mark.parametrize("V,M,d", [(30001, 24, 200), (17000, 33, 72), (40002, 64, 1032), (50000, 100, 192), (33333, 200, 72), (20000, 300, 520),
                                     (50001, 129, 64), (49409, 257, 192), (25000, 700, 128), (24577, 513, 1088),
                                     (30001, 16, 4104), (20000, 5, 4096), (40000, 1, 72), (17001, 12, 2056),
                                     (30001, 9, 2048), (30001, 13, 4096), (30001, 8, 2504), (28673, 7, 5000), (66001, 3, 2040), (30001, 2, 520),
                                     (24577, 11, 1544), (28001, 4, 512)])
def test_dense(V, M, d):
    W, H = _normal(3, V, d), _normal(4, M, d)
    logits = torch.full((M + 1, V), 7.0, dtype=torch.float32, device="cuda")
    B.nanospec_dense_head(W, H, V, d, M, logits[:M])
    _check(logits[:M], W, H, "dense")
    assert torch.all(logits[M] == 7.0)


@pytest.mark.parametrize("n", [0, 1, 257, 1000, 33000])
@pytest.mark.parametrize("M,d", [(100, 192), (100, 200), (129, 128), (300, 192), (300, 136), (300, 4096)])
def test_many_hidden_rows_on_a_long_list(M, d, n):
    """256 x 128 and 256 x 256 logits and head_gemm_kernel on gathered rows, and on the packed buffer, whose logits go to columns of their own"""
    V, window = 50000, 33000                                  # a capacity at which the larger blocks are taken
    W, H = _normal(5, V, d), _normal(6, 1, M, d)
    ids = np.sort(np.random.default_rng(n + M).permutation(V)[:n]).astype(np.int32)
    st = B.State(V, d, 1, window, 1, M, 1)
    B.nanospec_packed_enable(st.h)
    B.nanospec_vocab_init(st.h, dev_ids(ids), np.array([0, n], np.int32), None, np.zeros(2, np.int32))
    out = [torch.full((M + 1, st.capacity), 7.0, dtype=torch.float32, device="cuda") for _ in range(2)]
    B.nanospec_sparse_head(st.h, W, H, M, out[0][:M])
    B.nanospec_packed_gather(st.h, W)
    B.nanospec_packed_head(st.h, H, M, out[1][:M])
    for logits in out:
        _check(logits[:M, :n], W[torch.from_numpy(ids).long().cuda()], H[0], n)
        assert torch.all(logits[M] == 7.0)
    st.close()


@pytest.mark.parametrize("V,M,d", [(24600, 300, 192), (16400, 513, 64), (50000, 100, 192), (17000, 64, 72)])
def test_dense_on_operands_at_any_address(V, M, d):
    """operands that start between two 16-byte addresses: what fetches straight into LDS cannot take goes to the kernel beside it"""
    W, H = _normal(7, V * d + 8)[4:4 + V * d].view(V, d), _normal(8, M * d + 8)[4:4 + M * d].view(M, d)
    assert W.data_ptr() % 16 and H.data_ptr() % 16
    logits = torch.full((M + 1, V), 7.0, dtype=torch.float32, device="cuda")
    B.nanospec_dense_head(W, H, V, d, M, logits[:M])
    _check(logits[:M], W, H, "dense")
    assert torch.all(logits[M] == 7.0)
