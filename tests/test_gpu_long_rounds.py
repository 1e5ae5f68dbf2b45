"""The kernels that run rounds while more than 16 variables are left: the 29-bit kernel from the caller's words, after the
pass that serves two rounds, from planes and from integers, into planes and into words (of long tensors, with tables of more
than 2^16 rows); the long passes by row (with shorter tables); the rounds that bind table variables; and all of these side by side in instances that begin at different rounds.  Which of them a shape
runs is written beside it and checked against the library's own schedule.  Exact arithmetic: equality with the oracle,
or with the proof from the vector where that has been compared."""
import random

import numpy as np
import pytest
import torch

from tests.test_tlookup_plan import BOTH, FIRST, FIRST_TWO, GRID, NO_PASS, PAIR, R29, UNREAD

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
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    Sb = Tb[rows]
    return Sb, Tb, zk.vec_from_bytes(Sb), zk.vec_from_bytes(Tb), torch.from_numpy(rows.astype(np.int32)).cuda()


def _kinds(zk, logD, logN, K=1, from_ints=False):
    """What runs the rounds before the first of the last passes; of the 29-bit kernel also how the arrays arrive and leave."""
    rounds = [r for r in zk.zkmi_selftest_tlookup_plan(1 << logD, 1 << logN, K, from_ints)[1] if r[:2] != (GRID, UNREAD)]
    long = rounds[:[r[0] for r in rounds].index(GRID)]
    return [r[0] if r[0] != R29 else ("words" if r[2] else "planes", "words" if r[3] else "planes") for r in long]


@pytest.mark.parametrize("logD,logN,want", [
    (18, 16, [FIRST, ("words", "words")]),
    (20, 8, [FIRST_TWO, NO_PASS, PAIR]),
    (20, 17, [FIRST_TWO, NO_PASS, ("words", "words"), BOTH]),
    (21, 17, [FIRST_TWO, NO_PASS, ("words", "planes"), ("planes", "words"), BOTH]),
    (22, 17, [FIRST_TWO, NO_PASS, ("words", "planes"), ("planes", "planes"), ("planes", "words"), BOTH]),
    (20, 18, [FIRST, ("words", "words"), BOTH, BOTH]),
    (18, 18, [FIRST, BOTH]),
])
def test_single(zk, orc, logD, logN, want):
    assert _kinds(zk, logD, logN) == want
    Sb, Tb, S, T, idx = _instance(zk, logD, logN, 10 * logD + logN)
    seed = bytes([logD, logN]) * 16
    rc, proof, _ = orc.tlookup_prove(seed, Sb, Tb)
    assert rc == 0
    for call in (zk.tlookup_prove, zk.tlookup_prove_by_rows):
        rc, got, _ = call(seed, S, idx, T)
        assert rc == 0 and got == proof


def test_instances_that_begin_at_different_rounds(zk, orc):
    shapes = [(20, 6), (19, 4), (18, 16), (17, 16), (20, 17)]
    assert [_kinds(zk, d, n, K=5) for d, n in shapes] == [
        [FIRST_TWO, NO_PASS, PAIR], [FIRST_TWO, NO_PASS, PAIR], [FIRST, ("words", "words")], [FIRST],
        [FIRST_TWO, NO_PASS, ("words", "words"), BOTH]]
    made = [_instance(zk, d, n, 7 * d + n) for d, n in shapes]
    seed = random.Random(5).randbytes(32)
    rc, want, _ = orc.tlookup_multi_prove(seed, [m[0] for m in made], [m[1] for m in made])
    rc_g, got, _ = zk.tlookup_prove_multi(seed, [m[2] for m in made], [m[4] for m in made], [m[3] for m in made])
    assert rc == 0 and rc_g == 0 and got == want


@pytest.mark.parametrize("logD,logN,want", [
    (18, 10, [FIRST, ("words", "words")]),
    (20, 10, [FIRST_TWO, NO_PASS, PAIR]),
    (20, 16, [FIRST_TWO, NO_PASS, PAIR]),
])
def test_from_integers(zk, logD, logN, want):
    assert _kinds(zk, logD, logN, from_ints=True) == want
    g = torch.Generator(device="cuda")
    g.manual_seed(logD + logN)
    N, D = 1 << logN, 1 << logD
    tx = torch.arange(N, dtype=torch.int32, device="cuda") - N // 2
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, tx) == 0
    idx = torch.randint(0, N, (D,), generator=g, device="cuda", dtype=torch.int32)
    S = zk.Vec(D)
    S.data.copy_(T.data.index_select(1, idx.long()))
    seed = bytes([logD, logN, 3, 4]) * 8
    rc, proof, _ = zk.tlookup_prove(seed, S, idx, T)
    rc_i, from_ints, _ = zk.tlookup_prove_small(seed, tx[idx.long()].contiguous(), None, None, idx, T)
    assert rc == 0 and rc_i == 0 and from_ints == proof
