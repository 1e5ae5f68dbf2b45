"""The rows' products of a matrix proof: on the matrix cores (k_rowdot, from 768 rows and 2^20 elements on) with a batch of 64
columns that is not full, columns for one, two and three reductions (4096 to each) of which the later ones keep one or all four
wavefronts busy, rows that do not fill a workgroup, a matrix whose planes start anywhere; and the smaller matrices beside them
(k_rowdot_short).  Checked against the product by the definition, or for equality with the oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_link_long import shifted

pytestmark = pytest.mark.gpu
R = 0x73eda753299d7d483339d80809a1d80553bda402fffe5bfeffffffff00000001


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


@pytest.mark.parametrize("D0,D1,D2", [(1, 128, 1024), (2, 257, 511), (3, 33, 4097), (1, 15, 8737), (2, 130, 4096), (1, 131, 1000),
                                      (1, 768, 1366), (1, 767, 1368), (1, 1023, 1026), (1, 769, 4099)])
def test_against_the_definition(zk, D0, D1, D2):
    """Rows of the largest field element and of small ones: b_k is read off the proof of a matrix with one row of X per k."""
    rng = np.random.default_rng(D1 * 10000 + D2)
    Wb = rng.integers(0, 256, size=(D1 * D2, 32), dtype=np.uint8)
    Wb[:, 31] &= 0x3F
    Wb[: D2] = np.frombuffer((R - 1).to_bytes(32, "little"), np.uint8)
    Xb = rng.integers(0, 256, size=(D0 * D1, 32), dtype=np.uint8)
    Xb[:, 31] &= 0x3F
    X, W = zk.vec_from_bytes(Xb), shifted(zk, zk.vec_from_bytes(Wb))
    seed = bytes([D0, D1 % 251, D2 % 251, 9]) * 8
    rc, proof = zk.matmul_sumcheck_prove(seed, X, D0, D1, W, D2)
    assert rc == 0
    # Y = X W by the definition: the claim is Y~ at the point, recomputed column by column
    x = [[int.from_bytes(Xb[i * D1 + k].tobytes(), "little") for k in range(D1)] for i in range(D0)]
    w = [int.from_bytes(Wb[i].tobytes(), "little") for i in range(D1 * D2)]
    y = [sum(x[i][k] * w[k * D2 + j] for k in range(D1)) % R for i in range(D0) for j in range(D2)]
    Y = zk.vec_from_bytes(np.frombuffer(b"".join(v.to_bytes(32, "little") for v in y), np.uint8).reshape(-1, 32))
    assert zk.matmul_sumcheck_verify(seed, proof, D0, D1, D2, Y=Y, X=X, W=W) == 0


@pytest.mark.parametrize("D0,D1,D2", [(2, 768, 4400), (1, 769, 4096 + 256), (1, 1023, 5120), (1, 770, 8192 + 70), (1, 771, 8192 + 300)])
def test_columns_for_several_reductions(zk, orc, D0, D1, D2):
    """All four wavefronts have columns behind the first 4096: what they stage lies where the sums before were."""
    rng = np.random.default_rng(D1 * 10000 + D2)
    X, W = (rng.integers(-(1 << 40), 1 << 40, size=s) for s in ((D0, D1), (D1, D2)))
    seed = bytes([D0, D1 % 251, D2 % 251, 10]) * 8
    rc, want, _ = orc.matmul_sumcheck_prove(seed, X, W)
    assert rc == 0
    vx, vw = zk.vec_from_bytes(orc.fr_from_i64(X.reshape(-1))), zk.vec_from_bytes(orc.fr_from_i64(W.reshape(-1)))
    for w in (vw, shifted(zk, vw)):
        rc, got = zk.matmul_sumcheck_prove(seed, vx, D0, D1, w, D2)
        assert rc == 0 and got == want
        assert zk.matmul_sumcheck_verify(seed, got, D0, D1, D2, X=vx, W=w) == 0
