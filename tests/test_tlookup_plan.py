"""The schedule of the tlookup prover (what computes a round's sums, where it finds the arrays), walked on the host
without a GPU through the function the prover itself takes every decision from.  What is pinned here is what a launch
relies on: a round never has a source of S the library has no kernel for, integers are read only by the two kernels
written for them, a round reads the layout the round before it has written (words before every pass and before the
host's rounds), and every challenge is bound exactly once.  From a vector of field elements the first pass may serve
the first two rounds (FIRST_TWO, then NO_PASS: nothing launched), after which two variables are bound at once from the
caller's arrays.  Of long tensors with tables of up to 2^16 rows these rounds read the table's rows instead, from vectors
and from integers alike, and passes over two variables (PAIR) follow.  The rounds of the last 16 variables come up to three from one pass (GRID); the last six of a single
proof, three of each of several, are the host's (HOST)."""
import pytest

FIRST, R29, BOTH, FIRST_TWO, NO_PASS, HOST, GRID, PAIR = 0, 1, 2, 5, 6, 7, 8, 9
CALLER, INTS, WORDS, PLANES, UNREAD, ROWS = 0, 1, 2, 3, 4, 5
MAX_LAZY = 8  # folds in a row whose results stay unreduced in 29-bit planes


def _plan(zk, D, N, K=1, from_ints=False):
    rc, rounds = zk.zkmi_selftest_tlookup_plan(D, N, K, from_ints)
    return rc, rounds


def _check(rounds, n, h, K, from_ints=False):
    """Follows the arrays through the rounds: what layout S and A are in, how many of the last challenges they (and the
    table's arrays) have yet to be bound to."""
    host = 6 if K == 1 else 3
    by_row = n >= 19 and n - h <= 16 and h >= 3
    from_ints = from_ints and not by_row
    layout, pending, pending_t, lazy = ROWS if by_row else INTS if from_ints else CALLER, 0, 0, 0
    left_in_pass = t_in_pass = 0
    on_host = False
    for k, (kind, src, a, b) in enumerate(rounds):
        left = n - k
        table = k >= h
        where = (n, h, K, from_ints, k)
        if on_host:
            assert (kind, src, a, b) == (HOST, UNREAD, 0, 0), where
            continue
        if left_in_pass:
            assert (kind, src, a, b) == (GRID, UNREAD, 0, 0), where
            left_in_pass -= 1
            continue
        if kind == NO_PASS:
            assert k == 1 and rounds[0][0] == FIRST_TWO and src == UNREAD and pending == 2
            continue
        assert src == layout, where
        if kind == HOST:
            assert layout in (CALLER, WORDS) and left <= host, where
            assert (a, b) == (0, pending + 8 * pending_t), where
            on_host = True
        elif kind == GRID:
            assert layout in (CALLER, WORDS) and host < left <= 16, where
            vars_, tvars = a % 8, a // 8
            assert b == pending + 8 * pending_t and pending <= 3, where
            assert 1 <= vars_ <= 3 and (left - vars_ - host) % 3 == 0, where  # all passes of a call end at the same places
            assert tvars == len([t for t in range(k, k + vars_) if t >= h]), where
            if pending:
                layout = WORDS
            pending, pending_t, left_in_pass = vars_, tvars, vars_ - 1
        elif kind == PAIR:
            assert by_row and k >= 2 and left > 16 and k + a <= h and 1 <= a <= 2, where
            assert b == pending + (8 if left - a <= 16 else 0) and pending == 2 and pending_t == 0, where
            layout = WORDS if b >= 8 else PLANES
            pending, left_in_pass = a, a - 1
        else:
            assert not by_row or kind == FIRST_TWO, where
            assert left > 16 or (from_ints and k < 2) or rounds[0][0] == FIRST_TWO and k < 2, where
            if kind == R29:
                assert not table and a == (layout != PLANES) and (1 << (left - 1)) > 256, where
                assert pending in (1, 2) and (pending == 1 or k == 2 and rounds[0][0] == FIRST_TWO), where
                lazy = 0 if b else lazy + pending
                assert lazy <= MAX_LAZY - 1, where
                layout = WORDS if b else PLANES
            elif kind == BOTH:
                assert table and k > 0 and pending == 1 and pending_t == (1 if k > h else 0), where
                layout = WORDS
            elif kind == FIRST:
                assert k == 0, where
            else:
                assert kind == FIRST_TWO and k == 0 and h >= 3 and n > 16 and not from_ints, where
            if kind in (R29, BOTH):
                assert pending == (2 if kind == R29 and k == 2 and rounds[0][0] == FIRST_TWO else 1), where
            pending, pending_t = (2 if kind == FIRST_TWO else 1), (1 if table else 0)
    assert left_in_pass == 0 and (on_host or n == 0)


def test_plan_of_the_shape_that_once_faulted():
    """D = 2^12, N = 2^4 from two integer columns: round 0 is the first-round kernel reading the integers, round 1 the
    29-bit kernel folding them into words, every later round reads the workspace."""
    import paper_2404_16109_amd as zk
    rc, rounds = _plan(zk, 1 << 12, 1 << 4, from_ints=True)
    assert rc == 12
    assert rounds[0][:2] == (FIRST, INTS)
    assert rounds[1] == (R29, INTS, 1, 1)
    # ten variables left: a pass over one, a pass over three, six for the host
    assert rounds[2] == (GRID, WORDS, 1, 1) and rounds[3] == (GRID, WORDS, 3, 1) and rounds[6] == (HOST, WORDS, 0, 3)
    assert [r[0] for r in rounds] == [FIRST, R29] + [GRID] * 4 + [HOST] * 6
    _check(rounds, 12, 8, 1, True)
    # the same shape from a vector: passes over three variables from the start; the first leaves the arrays as they are
    rc, from_vec = _plan(zk, 1 << 12, 1 << 4)
    assert [r[0] for r in from_vec] == [GRID] * 6 + [HOST] * 6
    assert from_vec[0] == (GRID, CALLER, 3, 0) and from_vec[3] == (GRID, CALLER, 3, 3) and from_vec[6] == (HOST, WORDS, 0, 3)
    _check(from_vec, 12, 8, 1)


def test_plan_of_the_headline_shape_matches_the_bench_model():
    import bench
    import paper_2404_16109_amd as zk
    for from_ints in (False, True):
        rc, rounds = _plan(zk, 1 << 25, 1 << 16, from_ints=from_ints)
        assert rc == 25 and bench.rounds_by_row(1 << 25, 1 << 16)
        assert rounds[0][:2] == (FIRST_TWO, ROWS) and rounds[1][0] == NO_PASS
        # rounds 2 to 8 by passes over two variables, from the rows, then from planes, the last over one and into words
        assert [r[0] for r in rounds[2:9]] == [PAIR, GRID] * 3 + [PAIR]
        assert [r for r in rounds if r[0] == PAIR] == [(PAIR, ROWS, 2, 2), (PAIR, PLANES, 2, 2), (PAIR, PLANES, 2, 2), (PAIR, PLANES, 1, 10)]
        assert [r[0] for r in rounds[9:]] == [GRID] * 10 + [HOST] * 6
        assert rounds[9] == (GRID, WORDS, 1 + 8 * 1, 1) and rounds[10] == (GRID, WORDS, 3 + 8 * 3, 1 + 8 * 1)
        assert rounds[19] == (HOST, WORDS, 0, 3 + 8 * 3)
        _check(rounds, 25, 9, 1, from_ints)
    # twice as many rows: the 29-bit kernel's rounds
    rc, rounds = _plan(zk, 1 << 25, 1 << 17)
    assert rc == 25 and not bench.rounds_by_row(1 << 25, 1 << 17)
    assert [r[0] for r in rounds[:9]] == [FIRST_TWO, NO_PASS] + [R29] * 6 + [BOTH] and rounds[0][1] == CALLER
    assert rounds[2][2] == 1 and rounds[7][3] == 1 and all(r[3] == 0 for r in rounds[2:7])
    _check(rounds, 25, 8, 1)


def test_29_bit_rounds_are_those_of_the_bench_model():
    import bench
    import paper_2404_16109_amd as zk
    for n in range(0, 28):
        for l in range(0, n + 1):
            for from_ints in (False, True):
                rc, rounds = _plan(zk, 1 << n, 1 << l, from_ints=from_ints)
                if rc == n:
                    by_row = bench.rounds_by_row(1 << n, 1 << l)
                    assert by_row == (PAIR in [r[0] for r in rounds])
                    want = [] if by_row else bench.rounds_on_29_bits(1 << n, 1 << l, from_ints)
                    assert [k for k, r in enumerate(rounds) if r[0] == R29] == want, (n, l, from_ints)
                    assert from_ints or n == 0 or (rounds[0][0] == FIRST_TWO) == bench.first_two_rounds_share_a_pass(1 << n, 1 << l)


def test_where_passes_meet_what_runs_before_them():
    import paper_2404_16109_amd as zk
    # after the pass that serves two rounds: both variables bound on the way into the first pass, from the caller's S
    rounds = _plan(zk, 1 << 17, 1 << 3)[1]
    assert [r[0] for r in rounds[:3]] == [FIRST_TWO, NO_PASS, GRID] and rounds[2] == (GRID, CALLER, 3, 2)
    rounds = _plan(zk, 1 << 18, 1 << 3)[1]
    assert [r[0] for r in rounds[:4]] == [FIRST_TWO, NO_PASS, GRID, GRID] and rounds[2] == (GRID, CALLER, 1, 2)
    # after a 29-bit round, which leaves words although another could follow by its length
    rounds = _plan(zk, 1 << 18, 1 << 3, from_ints=True)[1]
    assert [r[0] for r in rounds[:3]] == [FIRST, R29, GRID] and rounds[1][2:] == (1, 1)
    # after a long pass, which may serve a round that a short one could; it leaves words
    rounds = _plan(zk, 1 << 19, 1 << 3)[1]
    assert [r[0] for r in rounds[:5]] == [FIRST_TWO, NO_PASS, PAIR, GRID, GRID]
    assert rounds[2] == (PAIR, ROWS, 2, 10) and rounds[4] == (GRID, WORDS, 3, 2)
    # after rounds that bind table variables
    rounds = _plan(zk, 1 << 19, 1 << 18)[1]
    assert [r[0] for r in rounds[:4]] == [FIRST, BOTH, BOTH, GRID] and rounds[3] == (GRID, WORDS, 1 + 8, 1 + 8)
    # the first round straight before a pass: nothing has been moved yet, S and T are the caller's
    rounds = _plan(zk, 1 << 17, 1 << 17)[1]
    assert rounds[0][0] == FIRST and rounds[1] == (GRID, CALLER, 1 + 8, 1 + 8)
    # several instances: three variables each are left to the host, however short they are
    rounds = _plan(zk, 1 << 5, 1 << 1, K=3)[1]
    assert rounds == [(GRID, CALLER, 2, 0), (GRID, UNREAD, 0, 0), (HOST, CALLER, 0, 2), (HOST, UNREAD, 0, 0), (HOST, UNREAD, 0, 0)]
    assert _plan(zk, 1 << 2, 1 << 1, K=3)[1] == [(HOST, CALLER, 0, 0), (HOST, UNREAD, 0, 0)]


def test_every_shape_has_something_for_every_round():
    import paper_2404_16109_amd as zk
    for n in range(0, 32):
        for l in range(0, n + 1):
            D, N = 1 << n, 1 << l
            for K in (1, 2, 8):
                rc, rounds = _plan(zk, D, N, K)
                assert rc == n
                _check(rounds, n, n - l, K)
            rc, rounds = _plan(zk, D, N, from_ints=True)
            takes_ints = zk.tlookup_small_workspace_bytes(D, N) == -(-zk.tlookup_workspace_bytes(D, N) // 256) * 256
            if rc < 0:
                # no integer path for this shape: tlookup_prove_small writes S out first and needs room for it
                assert rc == zk.ZK_E_BADARG and not takes_ints
                continue
            assert takes_ints and N <= 1 << 16 and D >= 4 * N and D > 1024
            if rounds[0][1] != ROWS:
                assert rounds[0][:2] == (FIRST, INTS) and rounds[1] == (R29, INTS, 1, 1)
                assert all(r[1] in (WORDS, UNREAD) for r in rounds[2:])
            _check(rounds, n, n - l, 1, True)


def test_plan_argument_errors():
    import paper_2404_16109_amd as zk
    assert _plan(zk, 1000, 8)[0] == zk.ZK_E_BADARG
    assert _plan(zk, 8, 16)[0] == zk.ZK_E_BADARG
    assert _plan(zk, 1 << 12, 1 << 4, K=2, from_ints=True)[0] == zk.ZK_E_BADARG
    assert _plan(zk, 1 << 12, 1 << 4, K=9)[0] == zk.ZK_E_BADARG
