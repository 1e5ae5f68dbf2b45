"""Verifications against all witness tensors, in which the evaluations' first stage and the leaves of m share a launch with the
leaves of A and B (csrc/tlookup_kernels.h, k_leaves_beside): one and several stages on either side, a table as long as the
tensor, leaves of m that do not fill a wavefront, vectors that no wide load can read, and more leaves than are
resident at once (2^24).  Every tensor altered by itself is rejected."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _inverses(zk, v, beta, stride):
    plus, out = zk.Vec(v.n), zk.Vec(v.n, stride)
    assert zk.fr_add_scalar(plus, v, beta) == 0 and zk.fr_batch_inverse(out, plus) == 0
    return out


@pytest.mark.parametrize("logD,logN,odd", [(12, 4, 0), (13, 0, 0), (13, 13, 1), (14, 6, 3), (16, 7, 0), (17, 14, 1), (18, 18, 0),
                                           (20, 15, 0), (22, 16, 1), (24, 10, 0)])
def test_every_tensor_is_read(zk, logD, logN, odd):
    D, N = 1 << logD, 1 << logN
    g = torch.Generator(device="cuda")
    g.manual_seed(64 * logD + logN)
    T = zk.Vec(N)
    assert zk.fr_from_i32(T, torch.randperm(N, generator=g, device="cuda").to(torch.int32) - N // 2) == 0
    idx = torch.randint(0, N, (D,), generator=g, device="cuda", dtype=torch.int32)
    S = zk.Vec(D, D + odd)
    S.data[:, :D] = T.data[:, :N].index_select(1, idx.long())
    seed = bytes([logD, logN]) * 16
    rc, proof, info = zk.tlookup_prove(seed, S, idx, T)
    assert rc == 0
    A, B = _inverses(zk, S, info["beta"], D + odd), _inverses(zk, T, info["beta"], N)
    m = torch.bincount(idx, minlength=N).to(torch.int32)
    check = lambda: zk.tlookup_verify(seed, proof, T, D, S=S, A=A, B=B, m=m)[0]
    assert check() == 0
    assert zk.tlookup_verify(seed, proof, T, D, A=A)[0] == 0
    assert zk.tlookup_verify(seed, proof, T, D, S=S, m=m)[0] == 0  # no leaves but those of m
    for v, n in ((S, D), (A, D), (B, N)):
        for at in (0, n - 1):
            v.data[1, at] ^= 1
            assert check() == zk.ZK_E_REJECT
            v.data[1, at] ^= 1
    for at in (0, N - 1):
        m[at] += 1
        assert check() == zk.ZK_E_REJECT
        m[at] -= 1
    assert check() == 0
