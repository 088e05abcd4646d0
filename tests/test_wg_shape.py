"""The rules that pick a launch's shape, evaluated on the host: what they pick for calls that every shape was measured on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
Q256, Q128, Q64_SPLIT, Q128_SPLIT = 1, 2, 3, 4  # FwdShape
TWO_LAUNCHES, B128, B64_SPLIT, B128_SPLIT, TWO_LAUNCHES_DQ128 = 0, 1, 2, 3, 4  # BwdShape


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    """pick([(launch, D, B, heads, T, H, W, s, group, pad), ...]) -> shapes"""
    exe = str(tmp_path_factory.mktemp("wg_shape") / "host_wg_shape_check")
    src = os.path.join(ROOT, "tests", "host_wg_shape_check.cpp")
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                           "-Wno-unused-command-line-argument", "-o", exe, src])

    def run(calls):
        text = "\n".join(" ".join(str(int(x)) if not isinstance(x, str) else x for x in c) for c in calls) + "\n"
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
        assert len(out) == len(calls)
        return [int(x) for x in out]

    return run


def dense(launch, D, units, n):
    return (launch, D, 1, units, 1, 1, n, 1, 0, 0)


def test_two_key_groups_only_while_the_large_shape_leaves_the_chip_idle(pick):
    """Splitting the keys pays while the 256-query shape has less than two rounds of workgroups; with more it lost 1 to 7 %."""
    few = [(1, 8190), (2, 12000), (1, 20160), (1, 32760), (8, 384), (24, 384)]
    assert all(x in (Q64_SPLIT, Q128_SPLIT) for x in pick([dense("fwd", D, *c) for c in few for D in (64, 128)]))
    assert pick([dense("fwd", 128, 4, 20160)]) == [Q128_SPLIT]
    many = [(20, 20160), (14, 30240), (10, 40320), (5, 80640), (63, 11340), (20, 8190), (40, 20160), (160, 20160)]
    assert all(x in (Q256, Q128) for x in pick([dense("fwd", D, *c) for c in many for D in (64, 128)]))
    # at six rounds and more Q256 is the better one at head_dim 128, Q128 at head_dim 64
    assert pick([dense("fwd", 128, *c) for c in many[:5] + many[6:]]) == [Q256] * 7
    assert pick([dense("fwd", 64, *c) for c in many]) == [Q128] * 8


def test_sixty_four_query_workgroups_only_in_one_round(pick):
    """A second round of them is slower than half as many large workgroups (34 units of 900 tokens: 33.5 us against 29)."""
    assert pick([dense("fwd", 128, *c) for c in ((34, 900), (33, 900), (55, 547), (29, 1061))]) == [Q256] * 4
    assert pick([dense("fwd", 128, *c) for c in ((16, 900), (28, 576), (24, 384))]) == [Q64_SPLIT] * 3


def test_one_round_of_the_large_shape_keeps_it_against_two_small_workgroups_a_cu(pick):
    """Measured 1 to 10 % faster in one round of 256-query workgroups than in twice as many of 128 queries, two on most CUs."""
    assert pick([dense("fwd", 128, *c) for c in ((192, 240), (84, 512), (225, 216), (152, 140), (148, 256), (48, 960))]) == [Q256] * 6
    assert pick([dense("fwd", 64, *c) for c in ((103, 377), (108, 384), (180, 140))]) == [Q256] * 3
    # where nearly all small workgroups are alone on their CUs, or the large ones would need another round, they stay
    assert pick([dense("fwd", 128, *c) for c in ((48, 390), (88, 280), (112, 144), (24, 2600), (48, 2600), (432, 64), (169, 1550))]) == [Q128] * 7


def test_classes_without_a_token_are_no_workgroups(pick):
    """Any-resolution grid on which only 2 of 16 classes hold a token: 2 x 64 units, not 16 x 64, decide (4-wavefront workgroups win)."""
    call = ("fwd", 64, 1, 64, 30, 2, 7, 4, 1, 1)
    assert pick([call]) == pick([dense("fwd", 64, 128, 30 * 2 * 4)])


def _classes(n, s, group):
    step = s if group else 1
    return [sum(1 for x in range(n) if x // step % s == p) for p in range(s)]


def test_gpu_tests_reach_every_shape(pick):
    """Every kernel that a launch can take, at both head_dims, plain and in the any-resolution mode, and each with a walk that wraps the ring
    of row offsets (more than 16 tiles of 64 rows a group), is taken by a test that compares it with the oracle: a refit of the tables that
    moves the calls of those tests elsewhere fails here."""
    import test_gpu_attention as fwd
    import test_gpu_bwd as bwd

    calls = [("fwd", D, 1, heads, 1, 1, n, 1, 0, 0) for D in (64, 128) for heads, n in fwd.WORKGROUP_SHAPES]
    calls += [("fwd", D, 1, heads, T, H, W, s, int(pattern == "group"), 1) for D in (64, 128) for heads, T, H, W, s, pattern in fwd.PADDED_SHAPES]
    calls += [("fwd", D, 1, 2, T, H, W, s, group, 1) for D in (64, 128) for T, H, W, s in fwd.PADDED_GROUPS for group in (0, 1)]
    calls += [("bwd", D, 1, heads, 1, 1, n, 1, 0, 0) for D in (64, 128) for heads, n in bwd.WORKGROUP_SHAPES + bwd.PAIR_SHAPES[D]]
    calls += [("bwd", 128, 1, heads, 1, 1, n, 1, 0, 0) for heads, n in bwd.LONG_SHAPES]
    calls += [("bwd", D, 1, heads, T, H, W, s, int(pattern == "group"), 1) for D in (64, 128) for heads, T, H, W, s, pattern in bwd.PADDED_SHAPES + bwd.PADDED_PAIR_SHAPES[D]]
    calls += [("bwd", D, B, heads, T, H, W, s, group, 1) for B, heads, D, T, H, W, s in bwd.PAD_CASES for group in (0, 1)]
    # a call that is one walk where it has the workspace reaches its shape only on the least one
    assert "skiparse_bwd_workspace_bytes" in bwd.LONG_WORKSPACES
    long = {("bwd", 128, 1, heads, 1, 1, n, 1, 0, 0) for heads, n in bwd.LONG_SHAPES}
    assert [c for c, walk in zip(calls, pick([("chain", *c[1:]) for c in calls])) if walk and c[0] == "bwd" and c not in long] == []
    met, wrapped = set(), set()
    for call, shape in zip(calls, pick(calls)):
        launch, D, _, _, T, H, W, s, group, pad = call
        largest = T * max(_classes(H, s, group)) * max(_classes(W, s, group)) if pad else T * H * W
        groups = 2 if shape in ((Q64_SPLIT, Q128_SPLIT) if launch == "fwd" else (B64_SPLIT, B128_SPLIT)) else 1
        met.add((launch, D, shape, pad))
        if (largest + 63) // 64 // groups > 16:
            wrapped.add((launch, D, shape, pad))
    want = {("fwd", D, shape, pad) for D in (64, 128) for shape in (Q256, Q128, Q64_SPLIT, Q128_SPLIT) for pad in (0, 1)}
    want |= {("bwd", D, shape, pad) for D in (64, 128) for shape in (TWO_LAUNCHES, TWO_LAUNCHES_DQ128, B128, B64_SPLIT, B128_SPLIT) for pad in (0, 1)}
    assert met == want
    # at head_dim 128 the four units of an any-resolution call take B64_SPLIT with 32 tiles at most
    assert wrapped == want - {("bwd", 128, B64_SPLIT, 1)}


def rows(row_bytes, n):
    return ("rows", row_bytes, 1, 1, 1, 1, n, 1, 0, 0)


def test_row_batches(pick):
    """A wavefront moves at most 4 KiB of rows in a batch, and rows above 768 B one by one: both measured slower than a wavefront a row."""
    sizes = list(range(16, 1024, 16))
    for n in (4608, 13824, 55296, 193536):
        for row_bytes, batch in zip(sizes, pick([rows(b, n) for b in sizes])):
            assert 1 <= batch <= 64
            assert batch == 1 or (row_bytes <= 768 and batch * row_bytes <= 4096 and n // batch >= 2048)
    assert pick([rows(b, 193536) for b in (16, 64, 128, 768, 784, 1008)]) == [64, 64, 32, 5, 1, 1]
    assert pick([rows(128, 2000)]) == [1]


def test_two_backward_launches_only_in_full_rounds(pick):
    """A launch of each kind in 256-owner workgroups is the better one in rounds that are full (or in one that mostly is), with long walks."""
    full = [(73, 12282), (192, 4584), (313, 5512), (48, 8190), (160, 20160), (6, 7844), (3, 17728)]
    assert all(x in (TWO_LAUNCHES, TWO_LAUNCHES_DQ128) for x in pick([dense("bwd", 128, *c) for c in full]))
    rest = [(20, 20160), (39, 5781), (414, 1824), (74, 385), (160, 960), (48, 400), (160, 2600), (12, 8190), (4, 20160)]
    assert pick([dense("bwd", 128, *c) for c in rest]) == [B128] * 9
    assert pick([dense("bwd", 128, *c) for c in ((1, 120), (8, 190), (24, 220), (1, 6116))]) == [B64_SPLIT] * 4
    assert pick([dense("bwd", 128, *c) for c in ((4, 2200), (1, 11191), (12, 1200))]) == [B128_SPLIT] * 3
    assert all(x in (TWO_LAUNCHES, TWO_LAUNCHES_DQ128) for x in pick([dense("bwd", 64, *c) for c in ((24, 2199), (7, 8474), (8, 6888))]))
    assert pick([dense("bwd", 64, *c) for c in ((160, 960), (572, 2563), (84, 14568))]) == [B128] * 3
    # units that a group of wavefronts has no tile in are never split
    assert all(x == B128 for x in pick([dense("bwd", D, u, n) for D in (64, 128) for u in (1, 40) for n in (1, 33, 64)]))


def test_bias_as_initial_accumulator_only_on_walks_that_hide_it(pick):
    """Any-resolution 8-bit calls: the bias of the keys starts every tile's logits where most tiles hold padding, and where there are tiles enough (slower by up
    to 10 % on 81 positions)."""
    def fp8(D, heads, T, H, W, s, group=0):
        return ("fp8", D, 1, heads, T, H, W, s, group, 1)

    short = [fp8(128, 40, 1, 21, 21, 3, 1), fp8(128, 34, 1, 25, 19, 3, 1), fp8(128, 40, 2, 13, 13, 2), fp8(128, 8, 7, 20, 13, 4, 1), fp8(64, 40, 2, 13, 13, 2), fp8(64, 24, 1, 25, 19, 3, 1)]
    assert pick(short) == [0] * 6
    long = [fp8(128, 20, 4, 13, 13, 2), fp8(128, 10, 21, 9, 13, 3), fp8(64, 20, 3, 13, 13, 2), fp8(64, 32, 9, 17, 21, 2, 1), fp8(64, 12, 21, 30, 45, 2)]
    assert pick(long) == [1] * 5
    few = [fp8(128, 40, 21, 45, 80, 2), fp8(64, 2, 1, 6, 258, 2)]  # whole lines at the end of long frames; the end of long lines
    assert pick(few) == [0] * 2


Q256_FULL, Q128_FULL = 5, 6  # FwdShape


def test_no_test_for_idle_wavefronts_where_none_is_idle(pick):
    """It costs up to 1.2 % there; at head_dim 64 it unbalances several rounds of units of 16 workgroups (40 x 4032: 4 %)."""
    full = {(48, 1536): Q128_FULL, (48, 1520): Q128_FULL, (15, 3584): Q256_FULL, (371, 128): Q128_FULL, (30, 2304): Q128_FULL}
    assert pick([dense("kernel", 128, *c) for c in full]) == list(full.values())
    assert pick([dense("kernel", 64, *c) for c in ((160, 384), (487, 128), (100, 4096), (40, 4032), (34, 4032), (80, 1984))]) == [Q128_FULL] * 6
    some = {(48, 1504): Q128, (160, 20160): Q256, (472, 480): Q128, (331, 96): Q128, (1, 32): Q128}
    assert pick([dense("kernel", 128, *c) for c in some]) == list(some.values())
    assert pick([dense("kernel", 64, *c) for c in ((1, 32), (40, 1984), (40, 3904), (60, 2368))]) == [Q128] * 4
    # the any-resolution mode always has the test
    assert pick([("kernel", 128, 1, 40, 21, 45, 80, 2, 0, 1), ("kernel", 64, 1, 4, 1, 9, 14, 2, 1, 1)]) == [Q256, Q128]


def test_gpu_tests_reach_the_kernels_with_and_without_that_test(pick):
    import test_gpu_attention as fwd

    met = {64: set(), 128: set()}
    for D in met:
        met[D] = set(pick([dense("kernel", D, *c) for c in fwd.WORKGROUP_SHAPES + fwd.LAST_WORKGROUPS]))
    assert all({Q256, Q128, Q256_FULL, Q128_FULL} <= m for m in met.values())


@pytest.mark.parametrize("launch,D,calls,want", [
    ("fwd", 128, [(1, 78), (35, 331), (49, 1465), (277, 1199), (141, 1997)], [Q128]),  # short units are not worth a merge; late rounds cost a full chip's clock
    ("fwd", 64, [(52, 276), (56, 244)], [Q128]),
    ("fwd", 128, [(3, 6151), (4, 3293), (10, 1512)], [Q64_SPLIT, Q128_SPLIT]),
    ("bwd", 128, [(2, 73), (7, 74), (17, 65), (1, 82)], [B128]),
])
def test_calls_timed_in_every_shape(pick, launch, D, calls, want):
    """Picks within 3 % of the best of all shapes, where the neighbouring ones measured up to 20 % slower."""
    assert set(pick([dense(launch, D, *c) for c in calls])) <= set(want)


def test_row_store_tests_reach_their_kernels(pick):
    """Every kernel with every kind of remainder, and with a last workgroup of few rows, on both sides of the lines at which rows are moved directly."""
    import test_gpu_row_stores as rows

    assert "skiparse_bwd_workspace_bytes" in [f.__name__ for f in rows.WORKSPACES]  # the shapes of "bwd" are those of the least workspace
    for cases, last in ((rows.FEW, rows.FEW_ROWS), (rows.KERNELS, rows.LAST)):
        for launch, D, kernel, units, before in cases:
            assert pick([dense(launch, D, units, before + n) for n in last]) == [kernel] * len(last), (launch, D, kernel)
    for launch, D, kernel, heads, W in rows.PADDED:
        assert pick([(launch, D, 1, heads, 1, 3, W + more, 2, 0, 1) for more in rows.LINES]) == [kernel] * len(rows.LINES), (launch, D, kernel)
    for D, kernel, heads, before in rows.LAYOUTS:
        calls = [("fwd", D, 1, heads, 1, H, W, 2, group, 0) for n in rows.LAST for H, W, group in ((2, 2 * (before + n), 0), (4, before + 4 * n, 1))]
        assert pick(calls[::2]) == [kernel] * len(rows.LAST) and kernel in pick(calls[1::2]), (D, kernel)
    both = {(launch, D, shape) for launch in ("kernel",) for D in (64, 128) for shape in range(1, 7)} | {("bwd", D, shape) for D in (64, 128) for shape in range(5)}
    assert {c[:3] for c in rows.KERNELS} == both
    # (128 queries a workgroup of the dQ launch: at head_dim 128 no any-resolution call of this size)
    assert {c[:3] for c in rows.PADDED} == {("fwd", D, shape) for D in (64, 128) for shape in range(1, 5)} | {("bwd", D, shape) for D in (64, 128) for shape in range(5)} - {("bwd", 128, 4)}
    fp8 = [("fp8", D, 1, 3, 1, 3, W, 2, 0, 1) for D in (64, 128) for W in rows.POSITIONS]
    assert pick(fp8[: len(fp8) // 2]).count(1) and pick(fp8[len(fp8) // 2 :]).count(1)


def test_one_walk_of_the_backward_where_its_rounds_are_full(pick):
    """0.82 to 0.98 of the time there, up to 1.87 on the others (timed both ways)."""
    full = [(160, 20160), (48, 8190), (64, 7960), (24, 8190), (16, 7961), (480, 960), (480, 1185), (64, 2907), (160, 1988), (320, 1780), (48, 4200), (64, 2315)]
    assert pick([dense("chain", 128, *c) for c in full]) == [1] * len(full)
    rest = [(48, 400), (8, 3000), (24, 1928), (12, 2807), (16, 2871), (48, 1780), (40, 2048), (40, 3000), (24, 2343), (12, 8116), (20, 20160), (160, 960), (160, 1017), (1, 120)]
    assert pick([dense("chain", 128, *c) for c in rest]) == [0] * len(rest)
    assert pick([("chain", 128, 1, 40, 21, 45, 80, 2, 0, 1), ("chain", 128, 1, 64, 30, 2, 7, 4, 1, 1), ("chain", 64, 1, 160, 1, 1, 20160, 1, 0, 0)]) == [1, 0, 0]


def test_queue_of_one_walk_hands_out_every_block_once(pick):
    """Whatever the units' number and the blocks', and however the workgroups are placed."""
    calls = [dense("queue", 128, units, n) for units in (1, 7, 8, 13, 20, 25, 48, 63, 160, 515) for n in (1, 256, 900, 2900, 7000, 8190, 20160)]
    assert all(pick(calls))


def test_gpu_tests_of_one_walk_are_given_to_it(pick):
    """All of them, units handed out 1 to 4 at a time, with and without a last group of fewer units, and chains of more workgroups than an XCD has CUs."""
    import test_gpu_bwd_chain as chain

    calls = [(128, B, heads, T, H, W, s, int(pattern == "group"), int(pad)) for B, heads, T, H, W, s, pattern, pad in chain.CASES]
    assert pick([("chain", *c) for c in calls]) == [1] * len(calls)
    together = pick([("queue", *c) for c in calls])
    units = [c[1] * c[2] * c[6] ** 2 for c in calls]
    assert set(together) == {1, 2, 3, 4} and {n for n, u in zip(together, units) if u % n} == {2, 3, 4}
    assert [c for c, n in zip(calls, together) if n == 1 and c[3] * c[4] * c[5] > 32 * 256]
