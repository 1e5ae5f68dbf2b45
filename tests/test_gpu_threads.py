"""Two host threads proving at the same time, each on a stream and a workspace of its own: the library's host state
(the pinned memory kernels report into, the channel a resident kernel reads its challenges from) is per thread, so
the proofs must come out as they do alone.  bench.py times this arrangement beside the headline."""
import random
import threading

import numpy as np
import pytest
import torch

from tests.pyref import R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(orc, zk, rng, D, N):
    T, seen = [], set()
    while len(T) < N:
        t = rng.randrange(R)
        if t not in seen:
            seen.add(t)
            T.append(t)
    rows = np.random.default_rng(rng.randrange(1 << 30)).integers(0, N, size=D)
    tb = orc.to_bytes(T)
    sb = tb[rows]
    return sb, tb, zk.vec_from_bytes(sb), zk.vec_from_bytes(tb), torch.from_numpy(rows.astype(np.int32)).cuda()


def test_two_threads_prove_at_once(zk, orc):
    rng = random.Random(4242)
    # two different lookups: one whose first pass serves two rounds, one that passes serve from the start
    cases = [_instance(orc, zk, rng, 1 << 17, 1 << 6), _instance(orc, zk, rng, 1 << 14, 1 << 9)]
    seeds = [rng.randbytes(32), rng.randbytes(32)]
    want = []
    for (sb, tb, _, _, _), seed in zip(cases, seeds):
        rc, proof, _ = orc.tlookup_prove(seed, sb, tb)
        assert rc == 0
        want.append(proof)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[], []]
    errors = []

    def worker(which):
        try:
            _, _, S, T, idx = cases[which]
            with torch.cuda.stream(streams[which]):
                for _ in range(6):
                    rc, proof, _ = zk.tlookup_prove(seeds[which], S, idx, T)
                    got[which].append((rc, proof))
        except Exception as e:  # surfaced below: a thread must not fail silently
            errors.append(repr(e))

    threads = [threading.Thread(target=worker, args=(w,)) for w in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for which in range(2):
        assert len(got[which]) == 6
        for rc, proof in got[which]:
            assert rc == 0 and proof == want[which]


def test_thread_state_can_be_made_and_given_back(zk, orc):
    """zkmi_thread_init allocates the calling thread's pinned state ahead of the first proof; zkmi_thread_release frees
    it, after which the next call allocates it again: proofs are the same before, between and after."""
    rng = random.Random(99)
    sb, tb, S, T, idx = _instance(orc, zk, rng, 1 << 13, 1 << 9)
    seed = rng.randbytes(32)
    rc, want, _ = orc.tlookup_prove(seed, sb, tb)
    assert rc == 0

    def worker(out):
        try:
            out.append(zk.zkmi_thread_init(1 << 9))
            out.append(zk.tlookup_prove(seed, S, idx, T)[:2])
            out.append(zk.zkmi_thread_release())
            out.append(zk.zkmi_thread_release())             # nothing left to free: still fine
            out.append(zk.tlookup_prove(seed, S, idx, T)[:2])  # allocates again by itself
            out.append(zk.zkmi_thread_release())
        except Exception as e:
            out.append(repr(e))

    got = []
    t = threading.Thread(target=worker, args=(got,))
    t.start()
    t.join()
    torch.cuda.synchronize()
    assert got == [0, (0, want), 0, 0, (0, want), 0]
    # the main thread's own state is untouched by another thread's release
    assert zk.tlookup_prove(seed, S, idx, T)[:2] == (0, want)


def test_thread_init_is_enough_for_a_full_batch(zk, orc):
    """After zkmi_thread_init(rows) no proof with tables of up to that many rows allocates: the staging buffer is where
    it was, also when all of a batch's tables are that long."""
    N, K = 1 << 16, zk.TLOOKUP_BATCH_MAX
    idx = torch.randint(0, N, (N,), dtype=torch.int32, device="cuda")
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, torch.arange(N, dtype=torch.int32, device="cuda")) == 0
    S = zk.Vec(N)
    S.data.copy_(T.data.index_select(1, idx.long()))
    torch.cuda.synchronize()
    got = []

    def worker():
        try:
            assert zk.zkmi_thread_init(N) == 0
            got.append(zk.zkmi_selftest_staging())
            got.append(zk.tlookup_prove_batch(b"\3" * 32, [S] * K, [idx] * K, [T] * K)[0])
            got.append(zk.zkmi_selftest_staging())
            got.append(zk.zkmi_thread_release())
            got.append(zk.zkmi_selftest_staging())
        except Exception as e:
            got.append(repr(e))

    t = threading.Thread(target=worker)
    t.start()
    t.join()
    torch.cuda.synchronize()
    assert len(got) == 5, got
    assert got[0][0] != 0 and got[1:] == [0, got[0], 0, (0, 0)], got


# Tables whose counts the host hashes and whose leaves' digests are handed over, and batches of either that cross the 64 leaves
# between the two (one of 2^13 rows, two of 2^12, four of 2^11)
@pytest.mark.parametrize("logN,K", [(3, 8), (10, 8), (11, 4), (11, 8), (12, 1), (12, 2), (12, 4), (13, 1), (13, 2), (13, 8), (14, 1), (14, 8)])
def test_thread_init_is_enough_for_short_tables(zk, logN, K):
    """The same at the lengths where counts or digests are staged, for proofs that are made, proofs that are refused while
    counting, and proofs whose earlier instances are looked through again once a later one is at fault."""
    N, D = 1 << logN, 1 << max(logN, 9)
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, torch.arange(N, dtype=torch.int32, device="cuda")) == 0

    def tensor(n):
        idx = torch.randint(0, N, (n,), dtype=torch.int32, device="cuda")
        S = zk.Vec(n)
        S.data.copy_(T.data[:, :N].index_select(1, idx.long()))
        return S, idx

    S, idx = tensor(D)
    bad, _ = tensor(D)
    bad.data.copy_(S.data[:, :D])
    bad.data[0, 3] ^= 1
    long_S, long_idx = tensor(1 << 19) if K > 1 else (None, None)
    torch.cuda.synchronize()
    got = []

    def worker():
        try:
            assert zk.zkmi_thread_init(N) == 0
            place = zk.zkmi_selftest_staging()
            assert place[0] != 0
            assert zk.tlookup_prove_batch(b"\3" * 32, [S] * K, [idx] * K, [T] * K)[0] == 0
            got.append(zk.zkmi_selftest_staging() == place)
            assert zk.tlookup_prove_batch(b"\3" * 32, [S] * (K - 1) + [bad], [None] * K, [T] * K)[0] == zk.ZK_E_NOT_IN_TABLE
            got.append(zk.zkmi_selftest_staging() == place)
            assert zk.tlookup_multiplicities(S, idx, T)[0] == 0
            got.append(zk.zkmi_selftest_staging() == place)
            if K > 1:
                rc, _, info = zk.tlookup_prove_multi(b"\3" * 32, [long_S] * (K - 1) + [bad], [long_idx] * (K - 1) + [idx], [T] * K)
                assert rc == zk.ZK_E_NOT_IN_TABLE and (info["bad_instance"], info["bad_index"]) == (K - 1, 3)
                got.append(zk.zkmi_selftest_staging() == place)
            assert zk.zkmi_thread_release() == 0
        except Exception as e:
            got.append(repr(e))

    t = threading.Thread(target=worker)
    t.start()
    t.join()
    torch.cuda.synchronize()
    assert got == [True] * (4 if K > 1 else 3), got
