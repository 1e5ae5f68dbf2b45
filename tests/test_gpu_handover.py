"""What kernels hand to the host through pinned memory: digest rows that one launch writes and a later one publishes,
and what a call leaves behind when it ends in an error that depends on data."""
import random

import numpy as np
import pytest
import torch

from tests.pyref import R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(zk, D, N, seed):
    rng = np.random.default_rng(seed)
    Tb = rng.integers(0, 256, size=(N, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    rows = rng.integers(0, N, size=D)
    Sb = Tb[rows]
    return Sb, Tb, zk.vec_from_bytes(Sb), zk.vec_from_bytes(Tb), torch.from_numpy(rows.astype(np.int32)).cuda()


# 2^16 entries have 512 leaves: the table's few go to the host from the launch before the one that ends the tensor's tree
# and publishes.  The proofs alternate between instances, so that a row left over from the call before would show in the
# digest.
def test_short_tables_beside_long_tensors(zk, orc):
    made = [_instance(zk, 1 << 16, N, N) for N in (1 << 8, 1 << 5, 1 << 8)]
    seeds = [random.Random(i).randbytes(32) for i in range(len(made))]
    want = [orc.tlookup_prove(seed, m[0], m[1])[1] for m, seed in zip(made, seeds)]
    for _ in range(12):
        for m, seed, proof in zip(made, seeds, want):
            rc, got, _ = zk.tlookup_prove(seed, m[2], m[4], m[3])
            assert rc == 0 and got == proof


def test_several_trees(zk, orc):
    sets = [[_instance(zk, 1 << d, 1 << n, 100 * k + d) for d, n in ((19, 6), (16, 9), (12, 3))] for k in range(2)]
    seed = b"\x17" * 32
    want = [orc.tlookup_multi_prove(seed, [m[0] for m in s], [m[1] for m in s])[1] for s in sets]
    for _ in range(4):
        for s, proof in zip(sets, want):
            rc, got, _ = zk.tlookup_prove_multi(seed, [m[2] for m in s], [m[4] for m in s], [m[3] for m in s])
            assert rc == 0 and got == proof


def test_errors_that_depend_on_data_leave_the_stream_idle(zk):
    """include/zkmi.h: such calls synchronise the stream before they return."""
    D, N = 1 << 17, 1 << 8
    Sb, Tb, S, T, idx = _instance(zk, D, N, 3)
    bad = zk.Vec(D)
    bad.data.copy_(S.data)
    bad.data[:, 77] ^= 1
    minus_t = R - int.from_bytes(Tb[5].tobytes(), "little")
    zeros, out = zk.vec_from_bytes(np.zeros((1000, 32), dtype=np.uint8)), zk.Vec(1000)
    ws = torch.empty(zk.tlookup_workspace_bytes(D, N), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        calls = {"hinted": (zk.ZK_E_NOT_IN_TABLE, lambda: zk.tlookup_prove(b"\1" * 32, bad, idx, T, ws=ws)[0]),
                 "found": (zk.ZK_E_NOT_IN_TABLE, lambda: zk.tlookup_prove(b"\1" * 32, bad, None, T, ws=ws)[0]),
                 "denominator": (zk.ZK_E_ZERO_DENOM, lambda: zk.tlookup_prove(b"\1" * 32, S, idx, T, ws=ws, forced_beta=minus_t)[0]),
                 "inverse": (zk.ZK_E_ZERO_DENOM, lambda: zk.fr_batch_inverse(out, zeros))}
        for name, (code, call) in calls.items():
            for _ in range(10):
                assert call() == code, name
                assert stream.query(), name
