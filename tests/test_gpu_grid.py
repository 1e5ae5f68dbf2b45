"""Several rounds from one pass (csrc/grid_dev.h) where its cases meet: passes of one, two and three variables, the
table's variables beginning before, inside and after a pass, instances that join between two passes, the first pass
taking over from each of the kernels that run before it.  Exact arithmetic: equality with the oracle."""
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


def _instance(orc, zk, logD, logN, rng):
    N, D = 1 << logN, 1 << logD
    Tb = np.frombuffer(rng.randbytes(32 * N), dtype=np.uint8).reshape(N, 32).copy()
    Tb[:, 31] &= 0x3F
    rows = np.random.default_rng(rng.randrange(1 << 30)).integers(0, N, size=D)
    Sb = Tb[rows]
    return Sb, Tb, zk.vec_from_bytes(Sb), zk.vec_from_bytes(Tb), torch.from_numpy(rows.astype(np.int32)).cuda()


# 2^16: passes from the first round on; 2^17, 2^18: after the pass that serves two rounds (pending both), or after the
# rounds that bind a table variable; 2^19: after the 29-bit rounds
@pytest.mark.parametrize("logD,logN", [(13, 13), (14, 8), (15, 15), (16, 0), (16, 7), (17, 1), (17, 14), (17, 17), (18, 3),
                                       (18, 15), (18, 17), (19, 10)])
def test_single(zk, orc, logD, logN):
    rng = random.Random(100 * logD + logN)
    Sb, Tb, Sv, Tv, idx = _instance(orc, zk, logD, logN, rng)
    seed = rng.randbytes(32)
    rc, want, _ = orc.tlookup_prove(seed, Sb, Tb)
    rc_g, got, _ = zk.tlookup_prove(seed, Sv, idx, Tv)
    assert rc == 0 and rc_g == 0 and got == want


# lengths that differ by one, two and three variables, down to one element, and by everything
@pytest.mark.parametrize("shapes", [[(4, 2), (5, 5), (6, 1)], [(9, 3), (8, 8), (10, 6), (7, 0)], [(3, 3), (2, 1), (1, 1), (0, 0)],
                                    [(12, 4), (0, 0), (5, 2)], [(14, 3), (13, 9), (6, 6)], [(6, 6)] * 8])
def test_lengths_mixed(zk, orc, shapes):
    rng = random.Random(len(shapes) + 10 * sum(d for d, _ in shapes))
    made = [_instance(orc, zk, d, n, rng) for d, n in shapes]
    seed = rng.randbytes(32)
    rc, want, _ = orc.tlookup_multi_prove(seed, [m[0] for m in made], [m[1] for m in made])
    rc_g, got, _ = zk.tlookup_prove_multi(seed, [m[2] for m in made], [m[4] for m in made], [m[3] for m in made])
    assert rc == 0 and rc_g == 0 and got == want
