"""The field arithmetic on the matrix cores (csrc/mfma_dev.h) where it can go wrong: every split of the variables into
stages, outputs that do not fill a tile, strides that forbid wide loads, and the values at which digits, column sums and
the closing reduction are largest.  Exact arithmetic: equality with the oracle."""
import random

import numpy as np
import pytest
import torch

from tests.pyref import R

pytestmark = pytest.mark.gpu
EXTREMES = [0, 1, R - 1, R - 2, (1 << 254) - 1, 1 << 254, int("7f" * 32, 16) % R, int("80" * 32, 16) % R]


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def restrided(zk, v, stride):
    out = zk.Vec(v.n, stride)
    out.data.zero_()
    out.data[:, :v.n].copy_(v.data[:, :v.n])
    return out


@pytest.mark.parametrize("nvars", [1, 2, 3, 6, 7, 8, 9, 12, 13, 14, 18, 19])
@pytest.mark.parametrize("values", ["random", "extreme"])
def test_mle_eval(zk, orc, nvars, values):
    rng = random.Random(100 * nvars + len(values))
    n = 1 << nvars
    if values == "random":
        rows = np.random.default_rng(nvars).integers(0, 256, size=(n, 32), dtype=np.uint8)
        rows[:, 31] &= 0x3F                                        # below r
        point = [rng.randrange(R) for _ in range(nvars)]
    else:
        rows = orc.to_bytes(EXTREMES)[np.random.default_rng(nvars).integers(0, len(EXTREMES), size=n)]
        if nvars % 2:
            rows[:] = orc.to_bytes([R - 1])[0]
        point = [rng.choice([R - 1, 2, (R + 1) // 2, 0, 1]) for _ in range(nvars)]
    want = orc.to_ints(orc.mle_eval(rows, orc.to_bytes(point)))[0]
    v = zk.vec_from_bytes(rows)
    for vec in (v, restrided(zk, v, n + 1)):
        rc, got = zk.fr_mle_eval(vec, point)
        assert rc == 0 and got == want


@pytest.mark.parametrize("stride", [1, 3])
def test_mle_eval_of_one_element(zk, orc, stride):
    """No variables: the value is the element itself, and the call needs no workspace."""
    import ctypes
    for value in (0, 1, 5, R - 1):
        v = restrided(zk, zk.vec_from_bytes(orc.to_bytes([value])), stride)
        out = zk.binding.fr_t()
        rc = zk.raw().fr_mle_eval(ctypes.byref(out), v.c, None, 0, None, 0, None)
        assert rc == 0 and int.from_bytes(out, "little") == value
        assert zk.fr_mle_eval(v, []) == (0, value)
