"""The matrix product's sums and rounds where their paths meet: one row per workgroup and four (2048 rows on), row counts
that leave a workgroup short, fewer chunks than shares, lengths whose rounds are the host's alone, end in one resident
round, or take one, two and three passes.  Exact arithmetic: equality with the oracle."""
import random

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


@pytest.mark.parametrize("D0,D1,D2", [(1, 1, 1), (3, 64, 5), (7, 128, 16), (65, 129, 33), (130, 257, 100), (9, 2047, 70),
                                      (33, 2048, 300), (200, 2051, 257), (2, 5000, 3)])
def test_products(zk, orc, D0, D1, D2):
    rng = np.random.default_rng(D0 * 7 + D1 + D2)
    X = rng.integers(-(1 << 15), 1 << 15, size=(D0, D1)).astype(np.int16)
    W = rng.integers(-(1 << 15), 1 << 15, size=(D1, D2)).astype(np.int16)
    seed = bytes([D1 % 256]) * 32
    Xb, Wb = orc.fr_from_i64(X.reshape(-1)), orc.fr_from_i64(W.reshape(-1))
    rc, want, _ = orc.matmul_sumcheck_prove(seed, X, W)
    assert rc == 0
    rc, got = zk.matmul_sumcheck_prove(seed, zk.vec_from_bytes(Xb), D0, D1, zk.vec_from_bytes(Wb), D2)
    assert rc == 0 and got == want
    rc, got = zk.matmul_sumcheck_prove_i16(seed, torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda())
    assert rc == 0 and got == want


@pytest.mark.parametrize("d", [0, 1, 6, 7, 8, 9, 10, 11, 13, 16, 17, 18])
def test_rounds(zk, orc, d):
    rng = random.Random(d)
    n = 1 << d
    rows = np.frombuffer(rng.randbytes(64 * n), dtype=np.uint8).reshape(2, n, 32).copy()
    rows[:, :, 31] &= 0x3F
    claim = orc.to_ints(orc.fr_sum(orc.fr_mul(rows[0], rows[1])))[0]
    seed = rng.randbytes(32)
    rc, want, _ = orc.sumcheck_prove_product(seed, rows[0], rows[1], orc.to_bytes([claim])[0])
    assert rc == 0
    rc, got = zk.sumcheck_prove_product(seed, zk.vec_from_bytes(rows[0]), zk.vec_from_bytes(rows[1]), claim)
    assert rc == 0 and got == want
