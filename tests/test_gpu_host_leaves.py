"""Lookups whose vectors have few leaves in all: up to 32 of them are hashed by the host.  Sizes on both sides of that, of one
element to 32 leaves, with hints, without, as integers; verification of each; an element outside the table.  Equality with the
oracle."""
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


@pytest.mark.parametrize("logD,logN", [(0, 0), (1, 0), (2, 1), (6, 6), (7, 7), (8, 3), (10, 8), (11, 4), (11, 11), (12, 0), (12, 11)])
@pytest.mark.parametrize("hints", [True, False])
def test_few_leaves(zk, orc, logD, logN, hints):
    rng = np.random.default_rng(64 * logD + 2 * logN + hints)
    Tb = rng.integers(0, 256, size=(1 << logN, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    S, T = zk.vec_from_bytes(Tb[rows]), zk.vec_from_bytes(Tb)
    idx = torch.from_numpy(rows.astype(np.int32)).cuda() if hints else None
    seed = bytes([logD, logN] * 16)
    rc, want, _ = orc.tlookup_multi_prove(seed, [Tb[rows]], [Tb])
    assert rc == 0
    for _ in range(2):  # the second finds the first one's bytes in the host's memory
        rc_g, got, _ = zk.tlookup_prove_multi(seed, [S], [idx], [T])
        assert rc_g == 0 and got == want
    assert zk.tlookup_verify_multi(seed, got, [T], [1 << logD])[0] == 0
    other = orc.tlookup_multi_verify(bytes(32), got, [Tb], [1 << logD])  # of one element and one row, the digests bind nothing
    assert zk.tlookup_verify_multi(bytes(32), got, [T], [1 << logD])[0] == other
    at = (1 << logD) - 1
    S.data[0, at] ^= 1
    rc_g, _, info = zk.tlookup_prove_multi(seed, [S], [idx], [T])
    assert rc_g == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == at


def test_no_bytes_stay_in_the_hosts_memory(zk):
    """The leaves are the caller's witness: none of their bytes is left in the staging buffer when a proof or a verification
    ends, accepted or not."""
    logD, logN = 11, 8
    rng = np.random.default_rng(5)
    D, N = 1 << logD, 1 << logN
    Tb = rng.integers(0, 256, size=(N, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    rows = rng.integers(0, N, size=D)
    S, T = zk.vec_from_bytes(Tb[rows]), zk.vec_from_bytes(Tb)
    idx = torch.from_numpy(rows.astype(np.int32)).cuda()

    seed = bytes([logD, logN] * 16)
    assert zk.zkmi_thread_init(1 << 12) == 0
    at, size = zk.zkmi_selftest_staging()
    assert size >= (D + N) * 32
    ctypes.memset(at, 0, (D + N) * 32)  # what other calls left
    left = lambda: np.count_nonzero(np.frombuffer(ctypes.string_at(at, (D + N) * 32), np.uint8))
    rc, proof, info = zk.tlookup_prove(seed, S, idx, T)
    assert rc == 0 and left() == 0
    A, B = zk.Vec(D), zk.Vec(N)
    for v, w in ((A, S), (B, T)):
        plus_beta = zk.Vec(w.n)
        assert zk.fr_add_scalar(plus_beta, w, info["beta"]) == 0 and zk.fr_batch_inverse(v, plus_beta) == 0
    assert zk.tlookup_verify(seed, proof, T, D, S=S, A=A, B=B)[0] == 0 and left() == 0
    A.data[0, 7] ^= 1
    assert zk.tlookup_verify(seed, proof, T, D, S=S, A=A, B=B)[0] == zk.ZK_E_REJECT and left() == 0
    S.data[0, D - 1] ^= 1
    assert zk.tlookup_prove(seed, S, idx, T)[0] == zk.ZK_E_NOT_IN_TABLE and left() == 0
