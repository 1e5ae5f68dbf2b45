"""The linking sumcheck's rounds served several at a time and on the host (csrc/grid_dev.h, csrc/zkattn_link.hip): passes of
one to three variables that lie before, across and behind the last row variable, rows shorter and longer than a
wavefront, shapes that are the host's after two rounds.  Exact arithmetic: equality with the oracle."""
import random

import pytest
import torch

from tests.test_gpu_link import make_witness, oracle_proof, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


@pytest.mark.parametrize("K", [1, 2, 3])
@pytest.mark.parametrize("log_rows,log_cols", [(0, 2), (2, 1), (1, 3), (3, 6), (9, 0), (0, 10), (8, 1), (2, 9), (7, 5), (10, 3),
                                               (6, 6), (4, 10), (12, 4), (3, 15)])
def test_proof(zk, orc, log_rows, log_cols, K):
    rows, cols = 1 << log_rows, 1 << log_cols
    w = make_witness(random.Random(100 * log_rows + 10 * log_cols + K), rows, cols, K, digit_bits=4, small_tables=rows * cols > 4096)
    seed = bytes([log_rows, log_cols, K, 1]) * 8
    rc, want, _ = oracle_proof(orc, seed, w, rows, cols)
    assert rc == 0
    Zp, X, Y, Yk, yhat, bases = to_device(zk, orc, w)
    rc, got = zk.zkattn_link_prove(seed, Zp, X, Y, Yk, yhat, bases, rows, cols)
    assert rc == 0 and got == want
