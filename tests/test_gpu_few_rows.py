"""Counting in tables of few rows (one launch up to 2^11 of them, m's leaves hashed by the host up to 64 in all) and A made by a
kernel of its own (up to 2^18 entries), on both sides of each limit, with repeated rows.  Exact: counts equal numpy's, proofs
the oracle's."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(zk, logD, logN, repeats=True):
    """(table bytes, rows, S, idx, T); with repeats the second half of the table is the first, backwards."""
    rng = np.random.default_rng(64 * logD + logN)
    D, N = 1 << logD, 1 << logN
    Tb = rng.integers(0, 256, size=(N, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    if repeats and N > 1:
        Tb[N // 2:] = Tb[:N // 2][::-1]
    rows = rng.integers(0, N, size=D)
    rows[D // 2:D // 2 + D // 8] = N - 1  # a long run
    return Tb, rows, zk.vec_from_bytes(Tb[rows]), torch.from_numpy(rows.astype(np.int32)).cuda(), zk.vec_from_bytes(Tb)


@pytest.mark.parametrize("logN", [0, 1, 2, 5, 6, 7, 10, 11, 12, 13, 14])
@pytest.mark.parametrize("repeats", [True, False])
def test_counts(zk, logN, repeats):
    Tb, rows, S, idx, T = _instance(zk, 14, logN, repeats)
    N = 1 << logN
    lowest = np.minimum(np.arange(N), N - 1 - np.arange(N)) if repeats else np.arange(N)
    want = np.bincount(lowest[rows], minlength=N)
    for hints in (idx, None):
        rc, m, _ = zk.tlookup_multiplicities(S, hints, T)
        assert rc == 0 and np.array_equal(m.cpu().numpy()[:N], want)
    S.data[3, 77] ^= 4
    for hints in (idx, None):
        rc, _, bad = zk.tlookup_multiplicities(S, hints, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and bad == 77


# rows 2^12 + 2^12: 64 leaves of m; one table more, or 2^14 rows, is beyond; long and short tables together
@pytest.mark.parametrize("shapes", [((12, 11),), ((13, 12),), ((13, 13),), ((14, 14),), ((12, 12), (13, 12)),
                                    ((12, 12), (13, 12), (11, 1)), ((13, 11), (14, 13), (3, 0))],
                         ids=lambda s: "+".join("%dx%d" % p for p in s))
@pytest.mark.parametrize("hints", [True, False])
def test_proofs(zk, orc, shapes, hints):
    parts = [_instance(zk, *s) for s in shapes]
    seed = bytes(range(32))
    rc, want, _ = orc.tlookup_multi_prove(seed, [p[0][p[1]] for p in parts], [p[0] for p in parts])
    assert rc == 0
    for _ in range(2):
        rc, got, _ = zk.tlookup_prove_multi(seed, [p[2] for p in parts], [p[3] if hints else None for p in parts],
                                            [p[4] for p in parts])
        assert rc == 0 and got == want


@pytest.mark.parametrize("logD,logN", [(12, 3), (17, 16), (18, 16), (18, 4), (19, 17)])
def test_a_made_apart(zk, orc, logD, logN):
    Tb, rows, S, idx, T = _instance(zk, logD, logN)
    seed = b"\x21" * 32
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    for call, hints in ((zk.tlookup_prove, idx), (zk.tlookup_prove, None), (zk.tlookup_prove_checked, idx),
                        (zk.tlookup_prove_by_rows, idx)):
        rc, got, _ = call(seed, S, hints, T)
        assert rc == 0 and got == want
    for at in (0, (1 << logD) - 1):
        S.data[2, at] ^= 1
        rc, _, info = zk.tlookup_prove(seed, S, idx, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == at
        S.data[2, at] ^= 1
    idx[5] = 1 << 30
    rc, _, info = zk.tlookup_prove(seed, S, idx, T)
    assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == 5


def test_no_counts_stay_in_the_hosts_memory(zk):
    _, _, S, idx, T = _instance(zk, 14, 12)
    assert zk.zkmi_thread_init(1 << 12) == 0
    at, size = zk.zkmi_selftest_staging()
    behind = 16 * 256 * 32  # the digests' rows
    assert size >= behind + 16 + (4 << 12)
    left = lambda: np.count_nonzero(np.frombuffer(ctypes.string_at(at + behind + 16, 4 << 12), np.uint8))
    ctypes.memset(at + behind, 0, 16 + (4 << 12))
    assert zk.tlookup_prove(bytes(32), S, idx, T)[0] == 0 and left() == 0
    assert zk.tlookup_multiplicities(S, idx, T)[0] == 0 and left() == 0
    S.data[0, 9] ^= 1
    assert zk.tlookup_prove(bytes(32), S, None, T)[0] == zk.ZK_E_NOT_IN_TABLE and left() == 0
