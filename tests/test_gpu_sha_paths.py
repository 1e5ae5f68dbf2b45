"""Which hash instructions the host uses is a choice of each call: proofs whose counts the host hashes (tables of up to 2^13
rows) while another thread asks for the portable compression function.  Exact: equality with the oracle."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zk():
    import paper_2404_16109_amd as zk
    assert torch.cuda.is_available()
    return zk


def _instance(zk, logD, logN):
    """(table bytes, rows, S, idx, T)"""
    rng = np.random.default_rng(64 * logD + logN)
    Tb = rng.integers(0, 256, size=(1 << logN, 32), dtype=np.uint8)
    Tb[:, 31] &= 0x3F
    rows = rng.integers(0, 1 << logN, size=1 << logD)
    return Tb, rows, zk.vec_from_bytes(Tb[rows]), torch.from_numpy(rows.astype(np.int32)).cuda(), zk.vec_from_bytes(Tb)


def test_another_thread_hashes_without_the_instructions(zk, orc):
    Tb, rows, S, idx, T = _instance(zk, 14, 12)
    seed = b"\x11" * 32
    rc, want, _ = orc.tlookup_prove(seed, Tb[rows], Tb)
    assert rc == 0
    done = threading.Event()

    def hash_on_and_off():
        data = bytes(20000)  # some 60 us without the instructions
        while not done.is_set():
            zk.zkmi_sha256(data, use_sha_instructions=False)

    other = threading.Thread(target=hash_on_and_off)
    other.start()
    try:
        got = [zk.tlookup_prove(seed, S, idx, T)[:2] for _ in range(200)]
    finally:
        done.set()
        other.join()
    assert [k for k, g in enumerate(got) if g != (0, want)] == []
