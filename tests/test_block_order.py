"""Direct pieces taken in blocks of two dimensions: when they are, and that
tables stay as long as the bytes need.  CPU: against the oracle through the
host interpreter, with a look at the plan.  GPU: the same layouts."""

import pytest

from paper_2211_05322_amd import binding as B
from tests import host_only
from tests.test_permuted_layouts import _gpu_run, host_perm_case


@pytest.fixture(scope="module")
def small_span(tmp_path_factory):
    """Parts of under 256 KiB a side, where the product's lie within 4 GiB."""
    return host_only.build(tmp_path_factory.mktemp("lib") / "small_span.so", RS_MAX_CHUNK_SPAN=1 << 18)


@pytest.fixture(scope="module")
def few_chunks(tmp_path_factory):
    """At most 1000 chunks a plan, where the product takes 2^24."""
    return host_only.build(tmp_path_factory.mktemp("lib") / "few_chunks.so", RS_MAX_DESCS=1000)


def noalloc_takes(p):
    """Whether the plan's tables fit reshard_execute_noalloc's scratch (its size check
    comes before any HIP call; the addresses are never used)."""
    try:
        B.reshard_execute_noalloc(p, [4096] * p.n_src, [4096] * p.n_dst, stream=0)
    except B.ReshardError as e:
        return e.status != B.RESHARD_EUNSUPPORTED
    return True


# sender pieces of 4 GiB and more on a side: shape, dtype, meshes and specs, permutations, chunk size
WIDE = [((1, 1 << 20, 64, 128), "bfloat16", (2,), "RS^0RR", (32,), "RRS^0R", None, (0, 2, 1, 3), 0),
        ((1, 1 << 20, 64, 128), "bfloat16", (2,), "RS^0RR", (32,), "RRS^0R", None, (0, 2, 1, 3), 1 << 20),
        ((1 << 27, 2, 16), "float32", (1,), "RRR", (1,), "RRR", None, (1, 0, 2), 0),
        ((13, 1, 34, 11100217), "float64", (1, 2), "S^1S^0RR", (2, 4), "RRRS^0", (3, 0, 2, 1), (0, 1, 3, 2), 1 << 18)]


@pytest.mark.parametrize("shape,dt,sm,ss,dm,ds,sp,dp,chunk", WIDE)
def test_chunks_of_wide_pieces_follow_the_chunk_size(shape, dt, sm, ss, dm, ds, sp, dp, chunk):
    p = B.reshard_plan(shape, dt, sm, ss, dm, ds, src_perm=sp, dst_perm=dp, chunk_bytes=chunk)
    st = B.reshard_plan_stats(p)
    # whole chunks of at least the automatic 16 KiB, and a rest per sender and receiver set
    assert st["n_descriptors"] <= 1.03 * st["bytes_read"] / max(chunk, 16384) + 4 * p.n_src * p.n_dst
    if chunk == 1 << 20:
        assert noalloc_takes(p)


# parts of several blocks, a short last part, rows left over, other outer levels;
# (tensor, the number of parts its largest piece is cut into)
PARTS = [(((2, 700, 16, 32), "float16", (2,), "RS^0RR", (1, 8), "RRS^1R", (0, 2, 1, 3)), 2),
         (((1, 640, 16, 64), "float32", (1,), "RRRR", (2, 8), "RRS^1R", (0, 2, 1, 3)), 10),
         (((1500, 3, 16), "float32", (1,), "RRR", (1,), "RRR", (1, 0, 2)), 2),
         (((3, 2, 1500, 3, 16), "float32", (1,), "RRRRR", (2,), "RRRRR", (1, 0, 3, 2, 4)), 3)]


@pytest.mark.parametrize("case,parts", PARTS)
@pytest.mark.parametrize("chunk", [0, 512, 3000])
def test_parts_of_wide_pieces_against_oracle(small_span, case, parts, chunk):
    shape, dt, sm, ss, dm, ds, dp = case
    with host_only.using(small_span) as lib:
        p = host_perm_case(shape, dt, sm, ss, None, dm, ds, dp, chunk_bytes=chunk)
        assert lib.test_blocked_chunks(p.handle) > 0
        # one chunk more at most per part, and per sender, receiver set and outer index for the rows left over
        st = B.reshard_plan_stats(p)
        c = max(256, (chunk or 4096) // 256 * 256)
        pieces = st["n_unit_tasks"] * 6
        assert st["n_descriptors"] <= st["bytes_read"] / c + pieces * (parts + 1)


# many pieces, each a few chunks longer in blocks
MANY = ("float16", (16,), "RS^0RR", (16,), "RRS^0R")


def test_table_within_the_noalloc_scratch_stays_in_it():
    dt, sm, ss, dm, ds = MANY
    p = B.reshard_plan((33, 496, 32, 128), dt, sm, ss, dm, ds, dst_perm=(0, 2, 1, 3), chunk_bytes=3968)
    assert B.reshard_plan_stats(p)["n_descriptors"] == 35072 and noalloc_takes(p)
    # the plain table would be too long as well: blocks stay
    q = B.reshard_plan((66, 496, 32, 128), dt, sm, ss, dm, ds, dst_perm=(0, 2, 1, 3), chunk_bytes=3968)
    assert B.reshard_plan_stats(q)["n_descriptors"] > 2 * 35072 and not noalloc_takes(q)


def test_plans_within_the_chunk_limit_stay_in_it(few_chunks):
    dt, sm, ss, dm, ds = "float16", (4,), "RS^0RR", (4,), "RRS^0R"
    with host_only.using(few_chunks) as lib:
        seen = set()
        for b in range(1, 6):  # 336 b chunks in blocks, 331 b in plain order
            args = (b, 124, 8, 128), dt, sm, ss
            try:
                p = host_perm_case(*args, None, dm, ds, (0, 2, 1, 3), chunk_bytes=1000)
            except B.ReshardError as e:
                assert e.status == B.RESHARD_EUNSUPPORTED and b >= 4
                seen.add("refused")
                continue
            assert "refused" not in seen
            blocked = lib.test_blocked_chunks(p.handle) > 0
            assert blocked or "blocked" in seen
            seen.add("blocked" if blocked else "plain")
            del p
        assert seen == {"blocked", "plain", "refused"}


# (tensor, devices on the two sides, the way back, in blocks, receiver sets in turn)
PATHS = [((2, 40, 16, 32), 2, (8, 2), False, False, False),    # 64-byte rows to 8 receivers
         ((2, 160, 16, 32), 2, (4, 2), False, True, False),    # to 4
         ((2, 80, 16, 64), 2, (8, 2), False, True, False),     # 128-byte rows to 8
         ((2, 16, 8, 1024), 2, (1, 4), False, False, False),   # blocks of 2 rows, 2 heads
         ((2, 16, 8, 1024), 2, (1, 2), False, True, False),    # 4 heads
         ((2, 16, 8, 512), 2, (1, 4), False, True, True),      # blocks of 4 rows; rows of heads 8 KiB apart
         ((2, 160, 64, 32), 2, (1, 4), False, True, True),     # 16 heads a set, one receiver
         ((2, 160, 64, 32), 2, (2, 4), False, True, False),    # ... two
         ((2, 160, 64, 32), 2, (2, 8), False, True, True),     # 8 heads a set, two receivers
         ((2, 130, 32, 64), 2, (2, 5), False, True, True),     # sets of 7 and 6 heads
         ((2, 128, 32, 64), 2, (2, 5), False, True, True),     # the last block whole
         ((2, 30, 96, 64), 1, (1, 2), True, True, False),      # the way back: blocks of heads
         ((2, 33, 130, 32), 2, (1, 3), True, True, False)]     # ... a rest of 1 head, of 65


@pytest.mark.parametrize("shape,n,dm,back,blocks,turns", PATHS)
def test_order_of_head_layouts(shape, n, dm, back, blocks, turns):
    a, b, perm = "RS^0RR", "RRS^1R", (0, 2, 1, 3)
    with host_only.using(host_only.plain()) as lib:
        if back:
            p = host_perm_case(shape, "float16", (1, n), b, perm, dm, "RS^1RR", None)
        else:
            p = host_perm_case(shape, "float16", (n,), a, None, dm, b, perm)
        assert (lib.test_blocked_chunks(p.handle) > 0, bool(lib.test_sets_in_turn(p.handle))) == (blocks, turns)
        del p


@pytest.mark.gpu
@pytest.mark.parametrize("shape,n,dm,back,blocks,turns", PATHS)
def test_gpu_order_of_head_layouts(shape, n, dm, back, blocks, turns):
    print(f"head layout {shape} {n} {dm} back={back}", flush=True)
    a, b, perm = "RS^0RR", "RRS^1R", (0, 2, 1, 3)
    if back:
        _gpu_run(shape, "float16", (1, n), b, perm, dm, "RS^1RR", None)
    else:
        _gpu_run(shape, "float16", (n,), a, None, dm, b, perm)


def test_units_to_two_receivers_leave_room_in_the_table():
    # 1-byte rows: slots of 16 of them, never a unit each
    p = B.reshard_plan((64, 200000, 2), "uint8", (4,), "RS^0R", (2, 2), "RRS^1")
    st = B.reshard_plan_stats(p)
    assert B.reshard_plan_unaligned_gather_chunks(p) > 0 and noalloc_takes(p)
    assert st["n_descriptors"] <= 1.1 * st["bytes_read"] / 4096 + 64 * 8
    # 129-byte rows, 9 units each: units while their table fits, else slots
    for rows, units in ((250000, True), (280000, False), (320000, True)):
        p = B.reshard_plan((2, rows, 258), "uint8", (2,), "RS^0R", (2, 2), "RRS^1", chunk_bytes=4096)
        assert (B.reshard_plan_unit_gather_chunks(p) > 0) == units, rows
        assert noalloc_takes(p) == (rows < 300000)
