"""The host-side rules of the dot calls (csrc/plan.h), compiled here without a GPU."""
import pytest

from planlib import SCRATCH, Plan


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return Plan(str(tmp_path_factory.mktemp("plan")))


def test_parts_are_lent_to_one_stream_only(plan):
    f = plan.L.lends
    assert f(0, 0, 5, 0, 0) == 1          # nobody's yet
    assert f(1, 5, 5, 0, 0) == 1
    assert f(1, 5, 6, 0, 0) == 0
    assert f(1, 0, 0, 0, 0) == 1          # the default stream
    for owned, of in ((0, 0), (1, 2)):
        assert f(owned, of, 2, 1, 0) == 0  # one handle, a stream in every thread
        assert f(owned, of, 2, 0, 1) == 0  # captured


def test_splits_stay_within_the_loop_the_cus_and_the_scratch(plan):
    f = plan.L.splits
    assert f(16, 1, 32, 1000, 1 << 25, 256) == 16
    assert f(2, 1, 32, 1000, 1 << 25, 256) == 32         # the loop's pieces
    assert f(2, 2, 80, 1000, 1 << 25, 256) == 80
    assert f(2, 1, 32, 1 << 20, 1 << 25, 256) == 8       # 32 MiB of u32 sums
    assert f(200, 1, 32, 1000, 1 << 25, 256) == 1
    assert f(2, 1, 32, 1000, 0, 256) == 1                # not lent
    assert f(2, 1, 32, 1 << 40, 1 << 25, 256) == 1


def test_rows_of_a_rotation_tile(plan):
    """The fewest rows at which all tiles run at once, a column tile's on one of 8 XCDs."""
    f = lambda rows, nt, vecs, cus=256: plan.L.tile_rows(rows, nt, vecs, cus)  # noqa: E731
    assert f(31, 8, 2) == 64 and f(247, 1, 2) == 64
    assert f(1024, 1, 2) == 64 and f(1025, 1, 2) == 128   # 32 CUs of one XCD: 16 tiles a vector
    assert f(1025, 1, 1) == 64 and f(2049, 8, 1) == 128
    assert f(2080, 8, 2) == 192 and f(2080, 9, 2) == 256
    assert f(104, 40, 1) == 64 and f(260, 40, 2) == 128
    assert f(200, 129, 2) == 256 and f(128, 65, 2) == 128 and f(128, 129, 2) == 256
    assert f(31, 8, 2, 8) == 256 and f(31, 8, 2, 16) == 64 and f(31, 8, 2, 0) == 256


def test_the_plan_and_the_launch_split_by_one_rule(plan):
    """One tile of 31 rows over 128 entries: 32 parts of the replicated loop, 16 of the Galois
    one; 20 tiles in 12 parts either way.  Three launches' costs and a part's of a tile."""
    assert plan.L.rot_splits(31, 128, 1, SCRATCH, 256, 0) == 32
    assert plan.L.rot_splits(31, 128, 1, SCRATCH, 256, 1) == 16
    for galois in (0, 1):
        assert plan.L.rot_cost(1, 31, 128, 1, SCRATCH, 256, galois) == 15 + 140 // (16 if galois else 32)
        assert plan.L.rot_splits(31, 1280, 2, SCRATCH, 256, galois) == 12
        assert plan.L.rot_cost(1, 31, 128, 1, 0, 256, galois) == 5 + 140         # not lent


def test_parts_of_a_loop_run_at_once(plan):
    """A column's parts run on one of 8 XCDs, 32 CUs: 6 row tiles x 10 columns x 2 vectors in 2
    parts are 20 columns, 3 on some XCDs, 36 workgroups there."""
    def at_once(rows, nt, vecs, parts):
        return -(-rows // 256) * vecs * -(-nt * parts // 8) <= 32

    assert plan.L.rot_splits(48 * 31, 1280, 2, SCRATCH, 256, 0) == 1
    assert plan.L.rot_splits(24 * 31, 1792, 2, SCRATCH, 256, 0) == 2
    for rows in (31, 260, 744, 1488, 2480):
        for nt in range(1, 129):
            for vecs in (1, 2):
                s = plan.L.rot_splits(rows, 128 * nt, vecs, SCRATCH, 256, 0)
                assert s == 1 or at_once(rows, nt, vecs, s), (rows, nt, vecs, s)


def test_columns_are_taken_apart_by_eights(plan):
    """A column tile's workgroups run on one of 8 XCDs: a first call of whole rounds has as many
    columns on each, or some XCDs go one round further (80 queries of 22 rotations, 7 row tiles x
    25 columns: 18 columns are 252 of 256 CUs' work, and 42 of 32 on two XCDs)."""
    for q, r, n, v, galois in ((80, 22, 3133, 2, 0), (72, 17, 6927, 1, 1), (46, 15, 9001, 2, 0), (20, 13, 70_016, 2, 1)):
        m = plan.L.first_cols(q, r, n, v, SCRATCH, 256, galois)
        assert m == n or m % 1024 == 0, (q, r, n)
    rot = list(range(-15, 16))
    for q, n, galois in ((48, 8879, True), (66, 5190, False), (80, 3133, False), (30, 10_836, False)):
        got = plan.plan(q, rot, n, 2, galois)
        assert got[1] == n or got[1] % 1024 == 0, (q, n)


def test_a_last_round_that_saves_little_is_not_taken_apart(plan):
    """8 tiles on each XCD's 32 CUs past the whole rounds take hardly longer than 8 alone."""
    assert plan.L.first_cols(80, 22, 3133, 2, SCRATCH, 256, 0) == 3133
    assert plan.plan(48, list(range(-15, 16)), 8879, 2, True) == (48, 8879)
    assert plan.plan(46, list(range(-15, 12)), 8293, 2, False) == (46, 8293)


def test_rounds_are_those_of_the_device(plan):
    """A last row tile goes apart up to 24 rounds of one tile per CU, however many CUs."""
    for cus in (32, 64, 256):
        assert plan.L.lead_tiles(260, 24 * cus, cus) == 1 and plan.L.lead_tiles(260, 24 * cus + 1, cus) == 2
    assert plan.L.lead_tiles(256, 100, 256) == 1 and plan.L.lead_tiles(385, 100, 256) == 2


def test_a_whole_loop_keeps_its_last_round(plan):
    """Not lent: 44 queries of 15 rotations against 23,261 entries, three tiles of rows and 182 of
    columns, are 2.1 rounds; the last 0.1 in a call of its own would wait for the rounds before it."""
    f = lambda q, r, n, v, scratch: plan.L.first_cols(q, r, n, v, scratch, 256, 0)  # noqa: E731
    assert f(44, 15, 23_261, 1, 0) == 23_261 and f(56, 26, 46_052, 1, 0) == 46_052
    assert f(44, 15, 23_261, 1, SCRATCH) < 23_261            # its loop splits: worth a call


def test_few_tiles_of_a_whole_loop_stay_on_the_rotation_kernel(plan):
    """Not lent, and all of its 64- or 128-row tiles at once: a tile of pairs takes longer than one of those."""
    rot = list(range(-15, 15))
    for q, n, galois in ((9, 632, True), (28, 1405, False), (16, 1000, False), (64, 64, True)):
        assert plan.plan(q, rot, n, 2, galois, scratch=0) == (0, 0), (q, n)
    assert plan.plan(64, rot, 5000, scratch=0)[0] == 64


def test_only_consecutive_lists_go_in_pairs(plan):
    rot = list(range(-15, 16))
    assert plan.plan(64, rot, 300_000) == (64, 299_008)
    assert plan.plan(64, rot, 300_000, scratch=0)[0] == 64                # captured: the same kernels, none split
    assert plan.plan(64, rot[::-1], 300_000) == (0, 0)
    assert plan.plan(64, rot[:26], 300_000) == (0, 0) and plan.plan(64, rot[:27], 300_000)[0] == 64
    assert plan.plan(64, rot[:-1] + [14], 300_000) == (0, 0)
    assert plan.plan(1, rot, 65_536) == (0, 0) and plan.plan(64, rot, 64) == (0, 0)
