"""Tables of equality weights on both sides of the length from which a thread makes sixteen entries
(csrc/poly.hip, kEqSharedVars).  Exact arithmetic: equality with the oracle."""
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


@pytest.mark.parametrize("nvars", [3, 4, 5, 7, 8, 9, 17, 18, 19])
@pytest.mark.parametrize("pad", [0, 5])
def test_lengths(zk, orc, nvars, pad):
    rng = random.Random(nvars)
    u = [rng.choice([0, 1, R - 1, rng.randrange(R), rng.randrange(R), rng.randrange(R)]) for _ in range(nvars)]
    n = 1 << nvars
    tab = zk.Vec(n, n + pad)
    tab.data.fill_(-1)
    assert zk.fr_eq_table(tab, u) == 0
    assert np.array_equal(zk.vec_to_bytes(tab), orc.eq_table(orc.to_bytes(u)))
    assert bool((tab.data[:, n:] == -1).all())


def test_a_long_table_is_no_chain_per_entry(zk):
    """2^22 entries cost a few products each, not one per variable: they take some 1.6 times as long as the elementwise
    product of two vectors of that length (ten times with a chain per entry; the line is between the two)."""
    nvars = 22
    u = [random.Random(1).randrange(R) for _ in range(nvars)]
    a, out = zk.Vec(1 << nvars), zk.Vec(1 << nvars)
    assert zk.fr_from_i32(a, torch.ones(1 << nvars, dtype=torch.int32, device="cuda")) == 0

    def best(call):
        times = []
        for _ in range(8):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            assert call() == 0
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop))
        return min(times)

    assert best(lambda: zk.fr_eq_table(out, u)) < 4 * best(lambda: zk.fr_mul(out, a, a))
