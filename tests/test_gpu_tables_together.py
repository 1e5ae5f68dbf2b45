"""Eight instances whose tables share launches: tables of one row to more than the counting's histograms take, with and
without hints, duplicate rows in some; the instance and index reported when an element is not in its table.  Equality with
the oracle."""
import numpy as np
import pytest
import torch

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
    if logN > 2:
        Tb[-2] = Tb[1]  # a duplicate
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    return Tb[rows], Tb, zk.vec_from_bytes(Tb[rows]), zk.vec_from_bytes(Tb), torch.from_numpy(rows.astype(np.int32)).cuda()


@pytest.mark.parametrize("shapes", [
    [(12, 12), (3, 0), (17, 17), (9, 1), (16, 8), (10, 10), (13, 7), (18, 16)],
    [(17, 17), (18, 17)],
    [(5, 2), (4, 4), (11, 3)]])
@pytest.mark.parametrize("hints", [True, False])
def test_instances(zk, orc, shapes, hints):
    made = [_instance(zk, d, n, 31 * d + n) for d, n in shapes]
    seed = bytes([len(shapes), hints] * 16)
    rc, want, _ = orc.tlookup_multi_prove(seed, [m[0] for m in made], [m[1] for m in made])
    idx = [m[4] for m in made] if hints else [None] * len(made)
    rc_g, got, _ = zk.tlookup_prove_multi(seed, [m[2] for m in made], idx, [m[3] for m in made])
    assert rc == 0 and rc_g == 0 and got == want
    # an element of the last but one instance that is not in its table
    at = len(made) - 2
    S = made[at][2]
    keep = S.data[0, 3].clone()
    S.data[0, 3] ^= 1
    rc_g, _, info = zk.tlookup_prove_multi(seed, [m[2] for m in made], idx, [m[3] for m in made])
    assert rc_g == zk.ZK_E_NOT_IN_TABLE and info["bad_instance"] == at and info["bad_index"] == 3
    S.data[0, 3] = keep
