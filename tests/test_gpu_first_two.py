"""The pass that serves the first two rounds, from vectors (k_round_first_two: tensors of 2^17 and 2^18 entries, tables of
more than 2^16 rows) and by row (k_first_two_rows): workgroups of 256 to 4096 positions, with and without a high weight
factor, vectors whose planes start anywhere.  Exact arithmetic: equality with the oracle, or a proof that the verifier accepts
against the tensor, whose evaluations are kernels of their own; by row also equality with the proof from the integers."""
import numpy as np
import pytest
import torch

from tests.test_gpu_link_long import shifted
from tests.test_tlookup_plan import CALLER, FIRST_TWO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


@pytest.mark.parametrize("logD,logN", [(17, 3), (17, 8), (18, 4)])
def test_against_the_oracle(zk, orc, logD, logN):
    assert zk.zkmi_selftest_tlookup_plan(1 << logD, 1 << logN, 1, False)[1][0][0] == FIRST_TWO
    rng = np.random.default_rng(logD * 100 + logN)
    Tb = rng.integers(0, 256, size=(1 << logN, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    Tb[0] = np.frombuffer((0x73eda753299d7d483339d80809a1d80553bda402fffe5bfeffffffff00000000).to_bytes(32, "little"), np.uint8)  # r - 1
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    rows[: 1 << (logD - 2)] = 0
    seed = bytes([logD, logN]) * 16
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    S, T = shifted(zk, zk.vec_from_bytes(Tb[rows])), zk.vec_from_bytes(Tb)
    rc, got, _ = zk.tlookup_prove(seed, S, torch.from_numpy(rows.astype(np.int32)).cuda(), T)
    assert rc == 0 and got == want


@pytest.mark.parametrize("logD,logN", [(21, 9), (22, 16), (23, 16), (24, 10)])
def test_against_the_integers(zk, logD, logN):
    g = torch.Generator(device="cuda")
    g.manual_seed(logD)
    N, D = 1 << logN, 1 << logD
    tx = torch.arange(N, dtype=torch.int32, device="cuda") - N // 2
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, tx) == 0
    idx = torch.randint(0, N, (D,), generator=g, device="cuda", dtype=torch.int32)
    S = zk.Vec(D, stride=D + 3)
    S.data[:, :D] = T.data.index_select(1, idx.long())
    seed = bytes([logD, logN, 3, 4]) * 8
    rc, proof, _ = zk.tlookup_prove(seed, S, idx, T)
    rc_i, from_ints, _ = zk.tlookup_prove_small(seed, tx[idx.long()].contiguous(), None, None, idx, T)
    assert rc == 0 and rc_i == 0 and from_ints == proof
    assert zk.tlookup_verify(seed, proof, T, D, S=S)[0] == 0


@pytest.mark.parametrize("logD,value,runs", [(23, 256, "everywhere"), (23, 65536, "everywhere"), (23, 65535, "everywhere"),
                                             (24, 256, "places"), (22, 256, "everywhere"), (23, -256, "everywhere")])
def test_tensors_of_one_value(zk, logD, value, runs):
    """Entries that are alike, in all four quarters of a workgroup's places: the sums over a place's four products are as
    large as they get (256 and 65536 have a digit -128 in the form vectors hold)."""
    N, D = 1 << 8, 1 << logD
    assert zk.zkmi_selftest_tlookup_plan(D, N, 1, False)[1][0][0] == FIRST_TWO
    g = torch.Generator(device="cuda")
    g.manual_seed(logD)
    tx = torch.arange(N, dtype=torch.int32, device="cuda") * 3 - N
    tx[7] = value
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, tx) == 0
    if runs == "everywhere":
        idx = torch.full((D,), 7, dtype=torch.int32, device="cuda")
    else:
        idx = torch.randint(0, N, (4, D >> 2), generator=g, device="cuda", dtype=torch.int32)
        idx[:, 4096 * 5:4096 * 45] = 7
        idx = idx.reshape(-1).contiguous()
    S = zk.Vec(D)
    S.data[:, :D] = T.data.index_select(1, idx.long())
    seed = bytes([logD, value & 0xFF, (value >> 8) & 0xFF, 5]) * 8
    rc, proof, _ = zk.tlookup_prove(seed, S, idx, T)
    rc_i, from_ints, _ = zk.tlookup_prove_small(seed, tx[idx.long()].contiguous(), None, None, idx, T)
    assert rc == 0 and rc_i == 0 and from_ints == proof
    assert zk.tlookup_verify(seed, proof, T, D)[0] == 0


@pytest.mark.parametrize("logD,logN,value", [(21, 17, None), (22, 18, None), (23, 17, 256), (23, 17, -256), (23, 17, 65535), (24, 17, 65536)])
def test_long_tables(zk, logD, logN, value):
    """The same from vectors: random entries, or runs of one value in all four quarters of a workgroup's places."""
    N, D = 1 << logN, 1 << logD
    assert zk.zkmi_selftest_tlookup_plan(D, N, 1, False)[1][0][:2] == (FIRST_TWO, CALLER)
    g = torch.Generator(device="cuda")
    g.manual_seed(logD)
    tx = torch.arange(N, dtype=torch.int32, device="cuda") * 3 - N
    if value is not None:
        tx[7] = value
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, tx) == 0
    idx = torch.randint(0, N, (4, D >> 2), generator=g, device="cuda", dtype=torch.int32)
    if value is not None:
        idx[:, :(D >> 2) - 4096 * 5] = 7
    idx = idx.reshape(-1).contiguous()
    S = zk.Vec(D, stride=D + 3)
    S.data[:, :D] = T.data.index_select(1, idx.long())
    seed = bytes([logD, logN, 6, (value or 0) & 0xFF]) * 8
    rc, proof, _ = zk.tlookup_prove(seed, S, idx, T)
    assert rc == 0 and zk.tlookup_verify(seed, proof, T, D, S=S)[0] == 0
    rc, by_rows, _ = zk.tlookup_prove_by_rows(seed, S, idx, T)
    assert rc == 0 and by_rows == proof
