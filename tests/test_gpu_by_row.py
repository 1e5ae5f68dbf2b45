"""Lookup proofs whose long rounds read the table's rows (csrc/tlookup_rows.h), at the lengths where their passes change:
one long pass (from rows to words, serving one round or two), two (through planes), three; rows found, checked beforehand,
while they are read, or against integers; wrong elements and row numbers, and which is reported.  Exact arithmetic:
equality with the oracle, or with the proof of the same statement that has been compared."""
import numpy as np
import pytest
import torch

from tests.test_tlookup_rows_plan import PAIR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(zk, logD, logN, seed):
    rng = np.random.default_rng(seed)
    Tb = rng.integers(0, 256, size=(1 << logN, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    Tb[0] = np.frombuffer((0x73eda753299d7d483339d80809a1d80553bda402fffe5bfeffffffff00000000).to_bytes(32, "little"), np.uint8)  # r - 1
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    rows[-(1 << (logD - 2)):] = 0
    S = zk.Vec(1 << logD, (1 << logD) + 3)
    T, idx = zk.vec_from_bytes(Tb), torch.from_numpy(rows.astype(np.int32)).cuda()
    S.data[:, :1 << logD] = T.data[:, :1 << logN].index_select(1, idx.long())
    return Tb, rows, S, T, idx


@pytest.mark.parametrize("logD,logN,passes", [(19, 3, 1), (19, 16, 1), (20, 16, 1), (21, 2, 2)])
def test_against_the_oracle(zk, orc, logD, logN, passes):
    plan = zk.zkmi_selftest_tlookup_rows_plan(1 << logD, 1 << logN)[1]
    assert len([r for r in plan if r[0] == PAIR]) == passes
    Tb, rows, S, T, idx = _instance(zk, logD, logN, 100 * logD + logN)
    seed = bytes([logD, logN]) * 16
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    for name, call in (("hints", lambda: zk.tlookup_prove(seed, S, idx, T)),
                       ("found", lambda: zk.tlookup_prove(seed, S, None, T)),
                       ("checked", lambda: zk.tlookup_prove_checked(seed, S, idx, T)),
                       ("rows", lambda: zk.tlookup_prove_by_rows(seed, S, idx, T))):
        rc, proof, _ = call()
        assert rc == 0 and proof == want, name


@pytest.mark.parametrize("logD,logN,pair", [(19, 16, True), (20, 8, False), (23, 16, True), (24, 12, True)])
def test_integers_and_the_verifier(zk, logD, logN, pair):
    D, N = 1 << logD, 1 << logN
    g = torch.Generator(device="cuda")
    g.manual_seed(logD)
    tx = torch.randint(-2**31, 2**31 - 1, (N,), generator=g, device="cuda", dtype=torch.int32)
    ty = torch.randint(-2**31, 2**31 - 1, (N,), generator=g, device="cuda", dtype=torch.int32) if pair else None
    T, Y = zk.Vec(N), zk.Vec(N)
    rho = 0x123456789abcdef0 << 180
    assert zk.fr_from_i32(T, tx) == 0
    if pair:
        assert zk.fr_from_i32(Y, ty) == 0 and zk.fr_axpy(T, T, rho, Y) == 0
    idx = torch.randint(0, N, (D,), generator=g, device="cuda", dtype=torch.int32)
    S = zk.Vec(D)
    S.data[:, :D] = T.data[:, :N].index_select(1, idx.long())
    x, y = tx[idx.long()].contiguous(), ty[idx.long()].contiguous() if pair else None
    seed = bytes([logD, logN, 7, 9]) * 8
    rc, proof, info = zk.tlookup_prove(seed, S, idx, T)
    rc_i, from_ints, _ = zk.tlookup_prove_small(seed, x, y, rho if pair else None, idx, T)
    assert rc == 0 and rc_i == 0 and from_ints == proof
    assert zk.tlookup_verify(seed, proof, T, D, S=S)[0] == 0
    for place in (0, D - 1, 3 * D // 4 + 65):
        wrong = x.clone()
        wrong[place] ^= 1
        rc, _, info = zk.tlookup_prove_small(seed, wrong, y, rho if pair else None, idx, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == place


def test_wrong_elements(zk):
    D = 1 << 19
    Tb, rows, S, T, idx = _instance(zk, 19, 6, 1)
    for places in ((D - 1,), (0,), (D // 2 + 3, D // 4 + 70, D - 2), (D // 4 - 1, D // 4)):
        bad, wrong = zk.Vec(D), idx.clone()
        bad.data.copy_(S.data[:, :D])
        for p in places:
            bad.data[5, p] ^= 1 << 9
            wrong[p] = 1 << 30
        for s, i in ((bad, idx), (S, wrong)):
            for call in (zk.tlookup_prove, zk.tlookup_prove_by_rows, zk.tlookup_prove_checked):
                rc, _, info = call(b"\x05" * 32, s, i, T)
                assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == min(places)
        rc, _, info = zk.tlookup_prove(b"\x05" * 32, bad, None, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and info["bad_index"] == min(places)


def test_the_first_instance_at_fault_is_reported(zk):
    """Instances of 2^19, 2^20 and 2^12 entries under one sumcheck: the longest's entries are read first, the shortest's
    while they are hashed."""
    parts = [_instance(zk, d, 4, d)[2:] for d in (19, 20, 12)]
    S, T, idx = [p[0] for p in parts], [p[1] for p in parts], [p[2] for p in parts]
    rc, proof, _ = zk.tlookup_prove_multi(b"\x07" * 32, S, idx, T)
    assert rc == 0
    assert zk.tlookup_verify_multi(b"\x07" * 32, proof, T, [s.n for s in S], S=S)[0] == 0
    for at_fault in ((0,), (1,), (2,), (0, 1), (1, 2), (0, 2), (0, 1, 2)):
        bad = []
        for i, s in enumerate(S):
            v = zk.Vec(s.n)
            v.data.copy_(s.data[:, :s.n])
            if i in at_fault:
                v.data[0, 77 + i] ^= 1
            bad.append(v)
        rc, _, info = zk.tlookup_prove_multi(b"\x07" * 32, bad, idx, T)
        assert rc == zk.ZK_E_NOT_IN_TABLE and (info["bad_instance"], info["bad_index"]) == (at_fault[0], 77 + at_fault[0])


# groups of 64 leaves: 675 (a lane per leaf), 803, 1154, 1476 (pairs of wavefronts), 1538 (a lane)
@pytest.mark.parametrize("logs", [(22, 20, 18), (22, 21, 18), (23, 20), (23, 21, 20, 19), (23, 22)], ids=str)
def test_digests_of_several_tensors(zk, logs):
    """The digests of A and B, made from rows by either kernel, are those of the vectors that a verification hashes."""
    N = 1 << 10
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(logs))
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, torch.arange(N, dtype=torch.int32, device="cuda") * 5 - N) == 0
    idx = [torch.randint(0, N, (1 << n,), generator=g, device="cuda", dtype=torch.int32) for n in logs]
    S = [zk.Vec(1 << n) for n in logs]
    for s, i in zip(S, idx):
        s.data[:, :s.n] = T.data[:, :N].index_select(1, i.long())
    rc, proof, info = zk.tlookup_prove_multi(b"\x09" * 32, S, idx, [T] * len(S))
    assert rc == 0

    def inverses(v):
        plus, out = zk.Vec(v.n), zk.Vec(v.n)
        assert zk.fr_add_scalar(plus, v, info["beta"]) == 0 and zk.fr_batch_inverse(out, plus) == 0
        return out

    A, B = [inverses(s) for s in S], [inverses(T)] * len(S)
    check = lambda: zk.tlookup_verify_multi(b"\x09" * 32, proof, [T] * len(S), [s.n for s in S], S=S, A=A, B=B)[0]
    assert check() == 0
    A[-1].data[2, A[-1].n - 1] ^= 1
    assert check() == zk.ZK_E_REJECT
