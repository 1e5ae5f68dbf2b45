"""Lookups on hosts with SHA instructions and without: proofs whose counts the host hashes (tables of up to 2^13 rows) while
another thread asks for the portable compression function, and every entry point on the way it goes without the instructions,
on both sides of 32 leaves of A and B and of 64 leaves of m.  Exact: equality with the oracle."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(zk, logD, logN):
    """(table bytes, rows, S, idx, T)"""
    rng = np.random.default_rng(64 * logD + logN)
    Tb = rng.integers(0, 256, size=(1 << logN, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    return Tb, rows, zk.vec_from_bytes(Tb[rows]), torch.from_numpy(rows.astype(np.int32)).cuda(), zk.vec_from_bytes(Tb)


def test_another_thread_hashes_without_the_instructions(zk, orc):
    Tb, rows, S, idx, T = _instance(zk, 14, 12)
    seed = b"\x11" * 32
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    done = threading.Event()

    def hash_on_and_off():
        data = bytes(20000)  # some 60 us without the instructions
        while not done.is_set():
            zk.zkmi_sha256(data, use_sha_instructions=False)

    other = threading.Thread(target=hash_on_and_off)
    other.start()
    try:
        got = [zk.tlookup_prove(seed, S, idx, T)[:2] for _ in range(200)]
    finally:
        done.set()
        other.join()
    assert [k for k, g in enumerate(got) if g != (0, want)] == []


@pytest.fixture
def portable(zk):
    assert zk.zkmi_selftest_without_sha_instructions(True) == 0
    yield
    assert zk.zkmi_selftest_without_sha_instructions(False) == 0


@pytest.mark.parametrize("logD,logN", [(0, 0), (1, 0), (6, 6), (8, 3), (9, 0), (9, 8), (10, 8), (11, 4), (11, 11), (12, 0), (13, 7),
                                       (14, 13), (14, 14), (18, 5), (19, 9)])
def test_without_the_instructions(zk, orc, portable, logD, logN):
    Tb, rows, S, idx, T = _instance(zk, logD, logN)
    D, seed = 1 << logD, bytes([logD, logN]) * 16
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    for name, call in (("hints", lambda: zk.tlookup_prove(seed, S, idx, T)), ("found", lambda: zk.tlookup_prove(seed, S, None, T)),
                       ("checked", lambda: zk.tlookup_prove_checked(seed, S, idx, T)),
                       ("rows", lambda: zk.tlookup_prove_by_rows(seed, S, idx, T))):
        for _ in range(2):
            rc, proof, _ = call()
            assert rc == 0 and proof == want, name
    assert zk.tlookup_verify(seed, want, T, D, S=S)[0] == 0
    rc, m, _ = zk.tlookup_multiplicities(S, idx, T)
    assert rc == 0 and np.array_equal(m.cpu().numpy()[:1 << logN], np.bincount(rows, minlength=1 << logN))
    for at in (0, D - 1):
        S.data[2, at] ^= 1
        rc, _, info = zk.tlookup_prove(seed, S, idx, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == at
        S.data[2, at] ^= 1


@pytest.mark.parametrize("logD,logN", [(9, 2), (10, 8), (12, 4), (15, 8)])
def test_integers_without_the_instructions(zk, orc, portable, logD, logN):
    D, N = 1 << logD, 1 << logN
    rng = np.random.default_rng(logD)
    tx, rows = rng.integers(-2**31, 2**31 - 1, size=N), rng.integers(0, N, size=D)
    Tb, seed = orc.fr_from_i64(tx), bytes([logD, 3]) * 16
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    x, idx = (torch.from_numpy(v.astype(np.int32)).cuda() for v in (tx[rows], rows))
    T = zk.vec_from_bytes(Tb)
    rc, proof, _ = zk.tlookup_prove_small(seed, x, None, None, idx, T)
    assert rc == 0 and proof == want
    x[D - 1] ^= 1
    rc, _, info = zk.tlookup_prove_small(seed, x, None, None, idx, T)
    assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == D - 1


@pytest.mark.parametrize("shapes", [((9, 3), (9, 9)), ((10, 8), (10, 2)), ((12, 4), (10, 8), (3, 0)), ((13, 13), (13, 12))],
                         ids=lambda s: "+".join("%dx%d" % p for p in s))
@pytest.mark.parametrize("hints", [True, False])
def test_several_without_the_instructions(zk, orc, portable, shapes, hints):
    parts = [_instance(zk, *s) for s in shapes]
    seed = b"\x44" * 32
    rc, want, _ = orc.tlookup_multi_prove(seed, [p[0][p[1]] for p in parts], [p[0] for p in parts])
    assert rc == 0
    S, idx, T = [p[2] for p in parts], [p[3] if hints else None for p in parts], [p[4] for p in parts]
    rc, got, _ = zk.tlookup_prove_multi(seed, S, idx, T)
    assert rc == 0 and got == want
    assert zk.tlookup_verify_multi(seed, got, T, [s.n for s in S], S=S)[0] == 0
    S[1].data[0, 5] ^= 1
    rc, _, info = zk.tlookup_prove_multi(seed, S, idx, T)
    assert rc == zk.ZK_E_NOT_IN_TABLE and (info["bad_instance"], info["bad_index"]) == (1, 5)


def test_a_verification_without_the_instructions(zk, portable):
    """All tensors given, few leaves and many."""
    for logD, logN in ((8, 4), (11, 8), (13, 9)):
        _, _, S, idx, T = _instance(zk, logD, logN)
        seed = b"\x55" * 32
        rc, proof, info = zk.tlookup_prove(seed, S, idx, T)
        assert rc == 0
        inverses = []
        for v in (S, T):
            plus, out = zk.Vec(v.n), zk.Vec(v.n)
            assert zk.fr_add_scalar(plus, v, info["beta"]) == 0 and zk.fr_batch_inverse(out, plus) == 0
            inverses.append(out)
        m = torch.bincount(idx, minlength=1 << logN).to(torch.int32)
        check = lambda: zk.tlookup_verify(seed, proof, T, 1 << logD, S=S, A=inverses[0], B=inverses[1], m=m)[0]
        assert check() == 0
        inverses[0].data[1, 7] ^= 1
        assert check() == zk.ZK_E_REJECT
