"""The linking sumcheck's long rounds (csrc/link_long.h), which start at 2^17 scores: rows of one entry to all of them, so
that row variables end before, inside and behind a pass and the low weight tables, one pass and two or three of them (from 2^19
scores on, 2^20 of integers, the later ones over arrays that were bound in place), one and two segments, vectors and integers
that allow no 16-byte loads, field elements over the whole range, integers at their largest.  Exact arithmetic: equality with the
oracle."""
import random

import numpy as np
import pytest
import torch

from tests.test_gpu_link import small_on_device, small_oracle_proof, small_witness, to_device
from tests.test_oracle_link import make_witness

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def shifted(zk, v):
    """The same vector where no plane starts at a multiple of four words."""
    out = zk.Vec(v.n, stride=v.n + 5)
    out.data = torch.empty(8 * (v.n + 5) + 1, dtype=torch.int32, device="cuda")[1:].view(8, v.n + 5)
    out.data[:, :v.n] = v.data[:, :v.n]
    return out


@pytest.mark.parametrize("log_rows,log_cols,K,aligned", [
    (17, 0, 2, True), (15, 2, 1, True), (12, 5, 2, False), (9, 8, 2, True), (7, 10, 1, False), (6, 11, 2, True), (5, 12, 2, True),
    (4, 13, 1, True), (1, 16, 2, True), (0, 17, 2, True), (10, 8, 2, True), (7, 11, 2, False),
    # the second pass starts at variable 2: rows end before it, where it starts, inside, behind it
    (1, 18, 1, True), (2, 17, 1, False), (3, 16, 1, True), (16, 3, 1, True),
    (0, 19, 2, True), (2, 17, 2, True), (3, 16, 2, False), (19, 0, 2, True), (5, 16, 1, True)])
def test_vectors(zk, orc, log_rows, log_cols, K, aligned):
    rows, cols = 1 << log_rows, 1 << log_cols
    rng = random.Random(1000 * log_rows + 10 * log_cols + K)
    w = make_witness(rng, rows, cols, K, digit_bits=4, small_tables=False)
    seed = rng.randbytes(32)
    to = orc.to_bytes
    rc, want, _ = orc.zkattn_link_prove(seed, to(w[0]), [to(a) for a in w[1]], to(w[2]), [to(a) for a in w[3]], to(w[4]), to(w[5]), rows, cols)
    assert rc == 0
    Zp, X, Y, Yk, yhat, bases = to_device(zk, orc, w)
    if not aligned:
        Zp, X, Y, Yk = shifted(zk, Zp), [shifted(zk, a) for a in X], shifted(zk, Y), [shifted(zk, a) for a in Yk]
    rc, got = zk.zkattn_link_prove(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == zk.ZK_OK and got == want
    # a relation broken in one entry
    for v in (Zp, X[-1], Y, Yk[0]):
        pos = rng.randrange(rows * cols)
        keep = v.data[0, pos].clone()
        v.data[0, pos] ^= 1
        assert zk.zkattn_link_prove(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)[0] == zk.ZK_E_REJECT
        v.data[0, pos] = keep


@pytest.mark.parametrize("log_rows,log_cols,K,out_bits,aligned", [
    (17, 0, 2, 30, True), (14, 3, 1, 32, True), (12, 5, 2, 30, False), (6, 11, 2, 16, True), (5, 12, 1, 16, False),
    (2, 15, 2, 30, True), (0, 17, 1, 20, True), (7, 11, 2, 29, True), (10, 9, 2, 30, False),
    # the second pass starts at variable 3
    (2, 18, 1, 32, True), (4, 16, 1, 20, False), (17, 3, 1, 30, True), (1, 19, 2, 30, True), (3, 17, 2, 29, False), (4, 16, 2, 30, True)])
def test_integers(zk, orc, log_rows, log_cols, K, out_bits, aligned):
    rows, cols = 1 << log_rows, 1 << log_cols
    gen = np.random.default_rng(100 * log_rows + log_cols + K)
    w = list(small_witness(gen, rows, cols, K, 8, out_bits))
    if out_bits >= 30:  # segment outputs at the largest that is accepted, side by side in all eight entries of a position
        top = (1 << out_bits) - 1 - (out_bits == 32)
        at = np.arange(8) * (rows * cols // 8) + 3
        w[3] = [np.minimum(a, top) for a in w[3]]
        for a in w[3]:
            a[at] = top
        w[2] = w[3][0] if K == 1 else w[3][0] * w[3][1]
        w[4] = [sum(int(v) for v in row) for row in w[2].reshape(rows, cols)]
    seed = bytes([log_rows, log_cols, K, out_bits]) * 8
    rc, want, _ = small_oracle_proof(orc, seed, w, rows, cols)
    assert rc == 0
    Zp, X, Y, Yk, yhat, bases = small_on_device(zk, orc, w)
    if not aligned:
        shift = lambda t: torch.cat([t[:1], t])[1:]
        Zp, X, Y, Yk = shift(Zp), [shift(a) for a in X], shift(Y), [shift(a) for a in Yk]
    rc, got = zk.zkattn_link_prove_small(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == zk.ZK_OK and got == want
    for t, rc_want in ((Zp, zk.ZK_E_REJECT), (X[0], zk.ZK_E_REJECT), (Y, zk.ZK_E_REJECT), (Yk[-1], zk.ZK_E_REJECT)):
        pos = int(gen.integers(0, rows * cols))
        keep = t[pos].clone()
        t[pos] = keep ^ 1
        assert zk.zkattn_link_prove_small(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)[0] == rc_want
        t[pos] = keep
    if K == 2:
        keep = Yk[0][5].clone()
        Yk[0][5] = 1 << 30
        assert zk.zkattn_link_prove_small(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)[0] == zk.ZK_E_BADARG
        Yk[0][5] = keep


def constant_output_tensors(log_rows, log_cols, value):
    """Two segments, the second of which has one output: Y^(2) is `value` everywhere."""
    import paper_2404_16109_amd as zk
    rows, cols = 1 << log_rows, 1 << log_cols
    D = rows * cols
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * log_rows + log_cols)
    X = [torch.randint(0, 1 << 16, (D,), generator=g, device="cuda", dtype=torch.int32), torch.zeros(D, dtype=torch.int32, device="cuda")]
    Yk = [torch.randint(0, 1 << 16, (D,), generator=g, device="cuda", dtype=torch.int32),
          torch.full((D,), value, dtype=torch.int32, device="cuda")]
    Y = Yk[0].long() * value
    canon = torch.zeros((rows, 4), dtype=torch.int64, device="cuda")
    canon[:, 0] = Y.reshape(rows, cols).sum(dim=1)
    yhat = zk.Vec(rows)
    assert zk.fr_from_canonical(yhat, canon) == 0
    return -X[0].long(), X, Y, Yk, yhat, [1, 1 << 16]


@pytest.mark.parametrize("log_rows,log_cols,value", [(13, 11, 256), (14, 10, 65536), (13, 11, 3)])
def test_vectors_of_one_value(zk, log_rows, log_cols, value):
    """From 2^24 scores on a workgroup takes 4096 positions; entries that are alike make the sums over a position's four
    products as large as they get.  The proof from the integers takes other sums first, and shorter ones after that."""
    rows, cols = 1 << log_rows, 1 << log_cols
    Zp, X, Y, Yk, yhat, bases = constant_output_tensors(log_rows, log_cols, value)
    seed = bytes([log_rows, log_cols, value & 0xFF, 7]) * 8
    rc, want = zk.zkattn_link_prove_small(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == zk.ZK_OK

    def vec(t):
        v = zk.Vec(t.numel())
        assert zk.fr_from_i32(v, t) == 0
        return v
    X, Yk = [vec(x) for x in X], [vec(y) for y in Yk]
    Zp, Y = zk.Vec(rows * cols), zk.Vec(rows * cols)
    assert zk.fr_mul_scalar(Zp, X[0], zk.synth.BLS12_381_R - 1) == 0 and zk.fr_mul(Y, Yk[0], Yk[1]) == 0
    rc, got = zk.zkattn_link_prove(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == zk.ZK_OK and got == want
    assert zk.zkattn_link_verify(seed, got, rows, cols, bases, yhat=yhat)[0] == zk.ZK_OK


def test_integers_of_one_value(zk):
    """From 2^27 scores on the second pass, over the folded arrays, has workgroups of 4096 positions."""
    rows, cols = 1 << 16, 1 << 11
    Zp, X, Y, Yk, yhat, bases = constant_output_tensors(16, 11, 256)
    seed = bytes([16, 11, 7, 8]) * 8
    rc, proof = zk.zkattn_link_prove_small(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == zk.ZK_OK
    assert zk.zkattn_link_verify(seed, proof, rows, cols, bases, yhat=yhat)[0] == zk.ZK_OK
