"""The schedule of lookup proofs whose long rounds read the rows of the table, walked on the host through the function the
prover takes it from: the first pass serves two rounds and reads rows, the pass after it binds both from the rows, every
later long pass binds the two variables of the one before from the planes that one has written, the last leaves words
for the short passes, and no long pass serves a variable of the table's."""
import pytest

from tests.test_tlookup_plan import CALLER, FIRST_TWO, GRID, HOST, NO_PASS, PLANES, UNREAD, WORDS

PAIR, ROWS = 9, 5


def test_every_shape():
    import paper_2404_16109_amd as zk
    for n in range(0, 32):
        for l in range(0, n + 1):
            for K in (1, 2, 8):
                rc, rounds = zk.zkmi_selftest_tlookup_rows_plan(1 << n, 1 << l, K)
                if n < 19 or l > 16 or n - l < 3:
                    assert rc == zk.ZK_E_BADARG
                    continue
                assert rc == n and rounds[0][:2] == (FIRST_TWO, ROWS) and rounds[1][:2] == (NO_PASS, UNREAD)
                k, source, pending, host = 2, ROWS, 2, 6 if K == 1 else 3
                while rounds[k][0] == PAIR:
                    _, src, served, b = rounds[k]
                    left = n - k
                    assert left > 16 and src == source and b % 8 == pending == 2
                    assert served == (1 if left == 17 and l == 16 else 2) and k + served <= n - l
                    assert (b >= 8) == (left - served <= 16)
                    if served == 2:
                        assert rounds[k + 1][:2] == (GRID, UNREAD)
                    k, source, pending = k + served, PLANES, served
                assert k > 2 and n - k <= 16
                left_in_pass = 0
                for k in range(k, n):
                    kind, src, a, b = rounds[k]
                    if left_in_pass:
                        assert (kind, src) == (GRID, UNREAD)
                        left_in_pass -= 1
                    elif kind == GRID:
                        assert src == WORDS and b % 8 == pending and n - k > host
                        pending, left_in_pass = a % 8, a % 8 - 1
                        assert a // 8 == len([t for t in range(k, k + a % 8) if t >= n - l])
                    else:
                        assert kind == HOST and (n - k < host or (n - k == host and b % 8 == pending))


def test_argument_errors():
    import paper_2404_16109_amd as zk
    for D, N, K in ((1000, 8, 1), (1 << 18, 1 << 4, 1), (1 << 20, 1 << 17, 1), (1 << 19, 1 << 4, 9), (1 << 32, 1 << 4, 1)):
        assert zk.zkmi_selftest_tlookup_rows_plan(D, N, K)[0] == zk.ZK_E_BADARG
