"""GPU parity of the stream initialisation at the sizes where its launches change: windows around the longest one that a
single workgroup takes, token segments and id ranges that end inside a workgroup, states that already hold another
stream (also one of the other policy), ids out of range, ragged batches.  Updates afterwards evict what the
initialisation left, so ring and counters are checked as well as the list."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2605_26444_amd import binding as B
from paper_2605_26444_amd import synth

from harness import csr, dev_ids

pytestmark = pytest.mark.gpu


def _tokens(V, seed, n):
    return synth.ZipfVocab(V, 1.1, seed).tokens(16, 0, n)


def _check(st, orc, what):
    got = st.read_active()
    for b, o in enumerate(orc):
        assert np.array_equal(got[b], o.active()), (what, b)


@pytest.mark.parametrize("policy", [B.POLICY_WINDOW, B.POLICY_FIFO])
@pytest.mark.parametrize("V,window,lengths,nT", [
    (1000, 64, [200, 63, 0], 16),
    (4097, 640, [640, 900], 64),
    (4096, 641, [641, 5000], 0),
    (32001, 1537, [1536 + (b & 1) for b in range(17)], 300),
    (16385, 1536, [1700 - b for b in range(18)], 100),
    (50001, 32768, [32768, 1], 128),
    (50001, 32769, [40000, 32769, 16384], 128),
    (128256, 40000, [39999, 70000], 2000),
    # around the longest prompts of one workgroup per sequence, and prompts of its range behind longer ones
    (30000, 256, [256], 40), (30000, 1024, [598], 40), (30000, 1024, [599], 40), (30000, 1024, [1500], 40),
    (30001, 2048, [1451 - (b & 1) for b in range(17)], 40), (30001, 2048, [1452 - (b & 1) for b in range(17)], 40), (30001, 4096, [2200 + b for b in range(17)], 40),
])
def test_init_over_any_earlier_state(policy, V, window, lengths, nT):
    nb = len(lengths)
    st = B.State(V, 64, nb, window, max(nT, 1), 1, 1)
    B.nanospec_set_stream_policy(st.h, policy)
    rng = np.random.default_rng(V + window)
    make = oracle.Vocab if policy == B.POLICY_WINDOW else oracle.FifoVocab
    for trial, keep in enumerate((1.0, 0.4, 1.0)):           # the second stream is shorter: parts of the first must be gone
        orc = [make(V, window) for _ in range(nb)]
        ctx = [_tokens(V, 7 * trial + b, int(n * keep)) for b, n in enumerate(lengths)]
        T = [rng.integers(0, V, nT).astype(np.int32) for _ in range(nb)]
        if trial == 2 and len(ctx[0]):
            ctx[0][:: max(1, len(ctx[0]) // 5)] = V            # ids out of range hold their place only
            T[0][:1] = -7
        f, o = csr(ctx)
        tf, to = csr(T)
        B.nanospec_vocab_init(st.h, dev_ids(f), o, dev_ids(tf), to)
        for b in range(nb):
            orc[b].init(ctx[b], T[b])
        _check(st, orc, (trial, "init"))
        assert (B.nanospec_last_device_error(st.h) == B.DEV_BAD_ID) == (trial == 2)
        for n in (5, 700, window // 2 + 3):                   # short (list patched), long, and one that evicts half the window
            new = [_tokens(V, 1000 + n + b, n) for b in range(nb)]
            f, o = csr(new)
            B.nanospec_vocab_update(st.h, dev_ids(f), o)
            for b in range(nb):
                orc[b].update(new[b])
            _check(st, orc, (trial, "update", n))
    st.close()


def test_init_after_the_other_policy():
    """what one policy leaves in the state must not show in a stream of the other"""
    V, window = 20000, 9000
    st = B.State(V, 64, 1, window, 8, 1, 1)
    for trial, (policy, n) in enumerate([(B.POLICY_FIFO, 12000), (B.POLICY_WINDOW, 3000), (B.POLICY_FIFO, 500), (B.POLICY_WINDOW, 11000),
                                         (B.POLICY_WINDOW, 100), (B.POLICY_FIFO, 9000), (B.POLICY_WINDOW, 9000)]):
        B.nanospec_set_stream_policy(st.h, policy)
        o = (oracle.Vocab if policy == B.POLICY_WINDOW else oracle.FifoVocab)(V, window)
        for call, (fn, n_ids) in enumerate([(None, n), (None, 0), ("u", 40), ("u", 2000), ("u", 9)]):
            ids = _tokens(V, 31 * trial + call, n_ids)
            if fn is None:
                B.nanospec_vocab_init(st.h, dev_ids(ids), [0, len(ids)], None, [0, 0])
                o.init(ids, [])
                if call == 0:                                 # keep the stream; the empty one comes second in odd trials only
                    _check(st, [o], (trial, call))
                    if trial % 2 == 0:
                        continue
                else:
                    _check(st, [o], (trial, call))
            else:
                B.nanospec_vocab_update(st.h, dev_ids(ids), [0, len(ids)])
                o.update(ids)
                _check(st, [o], (trial, call))
    st.close()


def test_init_recorded_in_a_graph():
    """a recorded initialisation is replayed over states that eager calls have changed, also under the other policy"""
    V, window, n = 30000, 33000, 34000
    for policy in (B.POLICY_WINDOW, B.POLICY_FIFO):
        for length in (n, 3000, 500):
            st = B.State(V, 64, 1, window, 8, 1, 1)
            B.nanospec_set_stream_policy(st.h, policy)
            ids = torch.from_numpy(_tokens(V, 3, length)).cuda()
            junk = dev_ids(_tokens(V, 4, 20000))
            run = lambda: B.nanospec_vocab_init(st.h, ids, [0, length], None, [0, 0])
            run()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                run()
            o = (oracle.Vocab if policy == B.POLICY_WINDOW else oracle.FifoVocab)(V, window)
            o.init(ids.cpu().numpy(), [])
            for replay in range(3):
                B.nanospec_vocab_update(st.h, junk, [0, 20000 if replay else 17])
                g.replay()
                _check(st, [o], (policy, length, replay))
            st.close()


@pytest.mark.parametrize("policy", [B.POLICY_WINDOW, B.POLICY_FIFO])
@pytest.mark.parametrize("n", [4094, 4096, 8191, 16384, 20478, 20480, 20490, 36863, 40000, 53248])
def test_patched_lists_of_several_passes(policy, n):
    """Appends that patch a list of n ids in place, 4096 entries to a pass and four passes read ahead of the one that is written: every step lets as many ids go as enter, at
    the list's ends, around the edges of passes and at random, alternately above and below each other so that runs of entries move both ways."""
    V, rng = 128256, np.random.default_rng(n)
    st = B.State(V, 64, 1, n, 16, 1, 1)
    B.nanospec_set_stream_policy(st.h, policy)
    orc = (oracle.Vocab if policy == B.POLICY_WINDOW else oracle.FifoVocab)(V, n)
    ids = np.sort(rng.choice(V, n, replace=False)).astype(np.int32)
    out = np.setdiff1d(np.arange(V, dtype=np.int32), ids)
    edges = [j for e in range(0, n + 1, 4096) for j in (e - 1, e, e + 1, e + 15) if 0 <= j < n]
    leave = list(dict.fromkeys([0, n - 1] + edges))
    leave = np.array(leave[:48] + [j for j in rng.permutation(n)[:80] if j not in set(leave)])
    ctx = np.concatenate([ids[leave], ids[np.setdiff1d(np.arange(n), leave)]])
    T = np.array([ids[0], out[-1]], np.int32)                  # one of them is in the window when it leaves
    f, o = csr([ctx])
    tf, to = csr([T])
    B.nanospec_vocab_init(st.h, dev_ids(f), o, dev_ids(tf), to)
    orc.init(ctx, T)
    for step, a in enumerate((16, 1, 7, 16, 2, 16, 15)):
        new = out[rng.integers(0, len(out), a)]
        if step == 1:
            new = out[:1]
        if step == 3:
            new = np.concatenate([out[-8:], out[1:9]])
        if step == 5:                                          # ids right beside the edges of passes
            new = out[np.clip(np.searchsorted(out, ids[np.array(edges)[rng.integers(0, len(edges), a)]]), 0, len(out) - 1)]
        f, o = csr([new])
        B.nanospec_vocab_update(st.h, dev_ids(f), o)
        orc.update(new)
        _check(st, [orc], (policy, n, step))
    assert B.nanospec_last_device_error(st.h) == 0
    st.close()
