"""Permuted local layouts (a buffer holds its shard as numpy.transpose(box,
perm)) and the tile-transpose chunks they need.

CPU: the planner's local shapes against the oracle's; the descriptor table
run on host memory (reshard_debug_execute_host, the kernel's tile and LDS
arithmetic with every access bounds-checked) against the oracle, bit for
bit, on seeded cases that span several tiles with ragged edges, every
element size, aligned and unaligned rows, and on argument errors.  GPU: the
kernels against the oracle on the same kinds of cases and on a transposed
activations at full size, every destination element compared, and seeded
permuted cases under random launch tunings.
"""

import random

import numpy as np
import pytest

import oracle
from paper_2211_05322_amd import binding as B
from tests import host_only
from tests.test_capi_host import run_host
from tests.test_oracle_pins import fmt_spec, random_dims

_NP = {"uint8": np.uint8, "float16": np.uint16, "float32": np.uint32, "float64": np.uint64}


def perm_cases(n, seed, big=False):
    """Random tensors (rows long enough for several 128-byte tiles), meshes,
    specs and a random permutation on each side."""
    rng = random.Random(seed)
    out = []
    while len(out) < n:
        ndim = rng.randint(2, 4)
        hi = 300 if big else 140
        shape = [rng.randint(1, 6) for _ in range(ndim)]
        for d in rng.sample(range(ndim), 2):  # two long dimensions
            shape[d] = rng.randint(20, hi)
        shape = tuple(shape)
        sm = tuple(rng.randint(1, 3) for _ in range(rng.randint(1, 2)))
        dm = tuple(rng.randint(1, 3) for _ in range(rng.randint(1, 2)))
        sp, dp = list(range(ndim)), list(range(ndim))
        rng.shuffle(sp)
        rng.shuffle(dp)
        if rng.random() < 0.2:
            sp = list(range(ndim))  # one side plain
        kw = {}
        if rng.random() < 0.4:
            kw["chunk_bytes"] = rng.choice([64, 1000, 8192, 40000])
        out.append((shape, rng.choice(list(_NP)), sm, fmt_spec(random_dims(rng, ndim, len(sm))), tuple(sp),
                    dm, fmt_spec(random_dims(rng, ndim, len(dm))), tuple(dp), kw))
    return out


def _inputs(shape, dt, sm, ss, sp, dm, ds, dp, seed):
    np_dtype = _NP[dt]
    es = np.dtype(np_dtype).itemsize
    rng = np.random.default_rng(seed)
    x = rng.integers(0, 256, size=int(np.prod(shape)) * es, dtype=np.uint8).view(np_dtype).reshape(shape)
    src = oracle.shard(x, sm, ss, sp)
    want = oracle.reshard(src, shape, sm, ss, dm, ds, src_perm=sp, dst_perm=dp)
    return src, want


def host_perm_case(shape, dt, sm, ss, sp, dm, ds, dp, seed=0, **kw):
    src, want = _inputs(shape, dt, sm, ss, sp, dm, ds, dp, seed)
    p = B.reshard_plan(shape, dt, sm, ss, dm, ds, src_perm=sp, dst_perm=dp, **kw)
    for k, w in enumerate(want):
        assert tuple(B.reshard_plan_local_shape(p, 1, k)) == w.shape
    for k, a in enumerate(src):
        assert tuple(B.reshard_plan_local_shape(p, 0, k)) == a.shape
    got = run_host(p, src, [w.shape for w in want], _NP[dt])
    for k, (g, w) in enumerate(zip(got, want)):
        assert np.array_equal(g, w), f"destination {k} differs"
    return p


@pytest.mark.parametrize("case", perm_cases(120, 77))
def test_host_permuted_against_oracle(case):
    shape, dt, sm, ss, sp, dm, ds, dp, kw = case
    host_perm_case(shape, dt, sm, ss, sp, dm, ds, dp, **kw)


@pytest.mark.parametrize("dt", list(_NP))
@pytest.mark.parametrize("shape", [(130, 70), (128, 64), (33, 517), (5, 200, 3), (2, 40, 300)])
def test_host_transpose_tiles(dt, shape):
    # the last two dimensions swapped on the destination side only: every
    # task is a tile transpose, with ragged tiles at the ends of both
    # dimensions (and whole tiles at 128 x 64)
    nd = len(shape)
    dp = tuple(range(nd - 2)) + (nd - 1, nd - 2)
    rep = "R" * nd
    p = host_perm_case(shape, dt, (2,), "S^0" + "R" * (nd - 1), None, (2,), rep, dp)
    assert B.reshard_plan_transpose_chunks(p) > 0


def test_host_transpose_unaligned_rows():
    # fp16 rows of 37 elements (74 bytes): no tile row starts on a 16-byte
    # boundary, and its vectors are loaded or stored where they lie
    for shape, dp in (((37, 90), (1, 0)), ((90, 37), (1, 0)), ((3, 37, 41), (2, 1, 0))):
        p = host_perm_case(shape, "float16", (1,), "R" * len(shape), None, (2,), "S^0" + "R" * (len(shape) - 1),
                           dp)
        assert B.reshard_plan_transpose_chunks(p) > 0


# extents at the edges of the transpose's tiles: rows or columns under 16
# bytes, one element past a tile, a last tile narrower than a vector, tiles
# that grow along one side, many small tiles in one chunk, columns on and off
# cache lines; (shape, bytes per element)
TILE_EDGES = [((3, 700), 1), ((700, 3), 1), ((9, 5, 7), 2), ((40, 9, 11), 8), ((2, 65, 513), 2), ((2, 513, 65), 2),
              ((1, 17, 4100), 1), ((1, 4100, 17), 1), ((1, 48, 2080), 2), ((300, 12, 20), 4), ((1, 2050, 2056), 2),
              ((1, 257, 1029), 1), ((1, 1031, 1040), 4)]
_TILE_DT = {1: "uint8", 2: "float16", 4: "float32", 8: "float64"}


@pytest.mark.parametrize("fan", [1, 3])
@pytest.mark.parametrize("shape,es", TILE_EDGES)
def test_host_transpose_tile_edges(shape, es, fan):
    nd = len(shape)
    dp = tuple(range(nd - 2)) + (nd - 1, nd - 2)
    p = host_perm_case(shape, _TILE_DT[es], (2,), "R" * (nd - 1) + "S^0", None, (fan, 2), "R" * (nd - 2) + "S^1R", dp)
    assert B.reshard_plan_transpose_chunks(p) > 0


# chunks larger than LDS takes at once loop over their tiles
TILE_LOOPS = [((1, 520, 1040), 2), ((300, 12, 20), 4), ((40, 9, 11), 8), ((1, 1030, 1290), 1), ((1, 520, 1040), 4),
              ((2, 131, 517), 4)]


@pytest.mark.parametrize("fan", [1, 4])
@pytest.mark.parametrize("shape,es", TILE_LOOPS)
def test_host_transpose_chunks_of_many_tiles(shape, es, fan):
    p = host_perm_case(shape, _TILE_DT[es], (1,), "RRR", None, (fan,), "RRR", (0, 2, 1), chunk_bytes=1 << 17)
    assert 0 < B.reshard_plan_transpose_chunks(p) <= -(-4 * shape[0] * shape[1] * shape[2] * es // (1 << 17))


# several tiles that LDS takes at once: 4-byte elements tile by tile (256 lanes
# and more of loads each), others and narrow tiles several to a pass
TILE_SETS = [((1, 520, 1040), 4, 1 << 14), ((2, 131, 517), 4, 1 << 14), ((1, 1040, 1040), 4, 1 << 14),
             ((3, 260, 33), 4, 1 << 15), ((2, 131, 517), 8, 1 << 14), ((2, 259, 517), 2, 1 << 15)]


@pytest.mark.parametrize("fan", [1, 2])
@pytest.mark.parametrize("shape,es,chunk", TILE_SETS)
def test_host_transpose_sets_of_tiles(shape, es, chunk, fan):
    p = host_perm_case(shape, _TILE_DT[es], (1,), "RRR", None, (fan,), "RRR", (0, 2, 1), chunk_bytes=chunk)
    assert B.reshard_plan_transpose_chunks(p) > 0


def test_transpose_table_follows_the_chunk_size():
    # 64 GiB in 256 KiB chunks: 2^18 of them, not one per LDS load
    p = B.reshard_plan((1, 1 << 16, 1 << 20), "uint8", (1,), "RRR", (1,), "RRR", dst_perm=(0, 2, 1), chunk_bytes=1 << 18)
    assert B.reshard_plan_transpose_chunks(p) == 1 << 18


# [batch, seq, head, dim] to [batch, head, seq, dim] and back: short and whole
# last blocks, rows that fit one block (plain order, all of the way back), rows
# a multiple of 4 KiB apart and not, one batch.  Which layouts are taken in
# blocks and in turns: test_block_order.py
HEADS = [((2, 80, 32, 64), "float16", (2,), (2, 2)), ((2, 64, 32, 64), "float16", (2,), (1, 4)),
         ((3, 70, 10, 40), "float16", (2,), (2, 2)), ((1, 300, 7, 16), "float32", (1,), (1, 2)),
         ((2, 33, 16, 64), "float16", (1,), (3, 2)), ((2, 130, 8, 128), "uint8", (2,), (1, 4))]


def heads_case(run, shape, dt, sm, dm, back):
    a, b = "RS^0RR", "RRS^1R"
    if back:
        return run(shape, dt, dm, b, (0, 2, 1, 3), sm, a, None)
    return run(shape, dt, sm, a, None, dm, b, (0, 2, 1, 3))


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("shape,dt,sm,dm", HEADS)
def test_host_heads(shape, dt, sm, dm, back):
    p = heads_case(host_perm_case, shape, dt, sm, dm, back)
    assert B.reshard_plan_transpose_chunks(p) == 0


# (bytes per element, receivers, the caller's cap, LDS reserved where the caller's cap is 20000 bytes)
@pytest.mark.parametrize("es,fan,cap,least", [(1, 1, 0, 27000), (2, 2, 0, 27000), (4, 1, 0, 0), (4, 2, 0, 0), (8, 2, 0, 0),
                                              (4, 3, 0, 27000), (8, 8, 0, 27000),
                                              (2, 1, -1, 0), (8, 8, -1, 0), (2, 1, 8, 20000)])
def test_transposes_keep_the_callers_cap(es, fan, cap, least):
    def lds(shape, cap):
        p = B.reshard_plan(shape, _TILE_DT[es], (1,), "RRR", (fan,), "RRR", dst_perm=(0, 2, 1), max_wgs_per_cu=cap)
        many = B.reshard_plan_transpose_chunks(p) >= 4096
        return many, lib.test_transpose_launch_lds(p.handle, 20000 if cap > 0 else 0)

    with host_only.using(host_only.plain()) as lib:
        for shape in ((1, 64, 64), (8, 4096, 4096)):
            many, own = lds(shape, -1)  # no cap: what the tiles take
            assert many == (shape[0] == 8) and 0 < own <= 32768
            assert lds(shape, cap)[1] == max(own, least if many or cap > 0 else 0)


# one of n destination parts has columns off 64-byte groups: stored through
# L2 when that is more than 1/7 of the tiles, 2/9 for 8-byte elements
@pytest.mark.parametrize("es,n,off,plain", [(2, 4, 0, False), (2, 8, 1, False), (1, 8, 1, False), (2, 5, 1, True),
                                            (4, 8, 1, False), (4, 5, 1, True), (8, 8, 1, False), (8, 5, 1, False),
                                            (8, 4, 1, True), (2, 8, 7, True), (2, 1, 1, True)])
def test_transpose_stores_by_the_share_of_parts(es, n, off, plain):
    with host_only.using(host_only.plain()) as lib:
        p = host_perm_case((1, n * (1088 // es) + off, 80), _TILE_DT[es], (1,), "RRR", None, (2, n), "RS^1R", (0, 2, 1))
        assert bool(lib.test_transpose_plain(p.handle)) == plain
        del p


# columns of 32-byte multiples off 64: plain, but for small tensors to one receiver
@pytest.mark.parametrize("shape,fan,plain", [((1, 2032, 80), 1, False), ((1, 2032, 80), 2, True), ((1, 2040, 80), 1, True),
                                             ((6, 2032, 2100), 1, True)])
def test_transpose_stores_of_half_groups(shape, fan, plain):
    with host_only.using(host_only.plain()) as lib:
        p = B.reshard_plan(shape, "float16", (1,), "RRR", (fan,), "RRR", dst_perm=(0, 2, 1))
        assert bool(lib.test_transpose_plain(p.handle)) == plain
        del p


# columns that follow one another in the buffer, off 64 bytes: their tiles are
# one run each, non-temporal up to 256 bytes a column or 4 receivers
@pytest.mark.parametrize("es,nb,na,fan,plain", [(2, 48, 400, 5, False), (8, 32, 5500, 5, False), (8, 33, 5500, 5, True),
                                                (8, 33, 5500, 4, False), (8, 39, 300, 8, True), (2, 61, 400, 5, False)])
def test_transpose_stores_of_dense_columns(es, nb, na, fan, plain):
    with host_only.using(host_only.plain()) as lib:
        p = host_perm_case((3, nb, na), _TILE_DT[es], (1,), "RRR", None, (fan,), "RRR", (0, 2, 1))
        assert bool(lib.test_transpose_plain(p.handle)) == plain
        del p


def test_permuted_outer_dims_need_no_transpose():
    # same innermost dimension on both sides, outer dimensions swapped: the
    # direct path with per-side strides, no tile transposes
    p = host_perm_case((6, 5, 64), "float32", (2,), "S^0RR", (1, 0, 2), (3,), "RS^0R", (0, 1, 2))
    assert B.reshard_plan_transpose_chunks(p) == 0


def test_identity_permutation_is_the_plain_plan():
    a = B.reshard_plan((8, 64, 96), "float16", (2, 2), "S^0RS^1", (2, 2), "RS^0S^1")
    b = B.reshard_plan((8, 64, 96), "float16", (2, 2), "S^0RS^1", (2, 2), "RS^0S^1", src_perm=(0, 1, 2),
                       dst_perm=(0, 1, 2))
    assert B.reshard_plan_stats(a) == B.reshard_plan_stats(b)
    assert B.reshard_plan_transpose_chunks(b) == 0


def test_permutation_errors():
    with pytest.raises(B.ReshardError) as e:
        B.reshard_plan((4, 4), "float16", (2,), "S^0R", (2,), "RS^0", dst_perm=(0, 0))
    assert e.value.status == B.RESHARD_EINVAL
    with pytest.raises(B.ReshardError) as e:
        B.reshard_plan((4, 4), "float16", (2,), "S^0R", (2,), "RS^0", src_perm=(0, 2))
    assert e.value.status == B.RESHARD_EINVAL
    with pytest.raises(B.ReshardError) as e:
        B.reshard_plan((4, 4), "float16", (2,), "S^0R", (2,), "RS^0", dst_perm=(1, 0),
                       flags=B.RESHARD_STRATEGY_SENDRECV)
    assert e.value.status == B.RESHARD_EUNSUPPORTED


# buffers above 4 GiB: a transpose piece must keep every tile within 32-bit
# offsets of its origin, cut along A or B (whichever stride makes the span
# too long) -- planning only here, the GPU tests below run them
BIG_TRANSPOSES = [((1, 70000, 70000), "uint8", None, (0, 2, 1)),
                  ((1, 40000, 60000), "float16", (0, 2, 1), None)]


@pytest.mark.parametrize("shape,dt,sp,dp", BIG_TRANSPOSES)
def test_transpose_pieces_above_4_gib_plan(shape, dt, sp, dp):
    p = B.reshard_plan(shape, dt, (1,), "RRR", (1,), "RRR", src_perm=sp, dst_perm=dp)
    assert B.reshard_plan_transpose_chunks(p) > 0
    assert B.reshard_plan_stats(p)["n_descriptors"] == B.reshard_plan_transpose_chunks(p)


def test_tile_strides_beyond_31_bits_take_the_element_path():
    # 128 destination rows of one tile would lie 34 MB apart: the planner
    # keeps such layouts off the transpose kernel (plain element pieces)
    p = B.reshard_plan((1, 200, 34000000), "uint8", (1,), "RRR", (1,), "RRR", src_perm=(0, 2, 1))
    assert B.reshard_plan_transpose_chunks(p) == 0
    st = B.reshard_plan_stats(p)
    assert st["bytes_written"] == 200 * 34000000 and st["n_descriptors"] > 0


def test_too_many_chunks_fails_cleanly():
    # 29 GB of bytes whose source and destination orders share no run and
    # whose strides keep them off the tile path: one chunk per few bytes,
    # far beyond the descriptor budget -- refused, and lowering stops there
    import time
    t = time.time()
    with pytest.raises(B.ReshardError) as e:
        B.reshard_plan((16, 8, 5298, 42608), "uint8", (2,), "RS^{0}RR", (3,), "RRRR",
                       src_perm=(0, 2, 3, 1), dst_perm=(2, 3, 1, 0))
    assert e.value.status == B.RESHARD_EUNSUPPORTED and "2^24" in str(e.value)
    assert time.time() - t < 60


# --------------------------------------------------------------------- GPU

def _gpu_run(shape, dt, sm, ss, sp, dm, ds, dp, seed=0, **kw):
    import torch
    from tests.test_gpu_parity import Guarded
    src, want = _inputs(shape, dt, sm, ss, sp, dm, ds, dp, seed)
    p = B.reshard_plan(shape, dt, sm, ss, dm, ds, src_perm=sp, dst_perm=dp, **kw)
    sb = []
    for a in src:
        g = Guarded(a.nbytes, 0xA5)
        if a.nbytes:
            g.body().copy_(torch.from_numpy(np.ascontiguousarray(a).reshape(-1).view(np.uint8).copy()))
        sb.append(g)
    db = [Guarded(w.nbytes, 0x5A) for w in want]
    B.reshard_execute(p, [g.ptr for g in sb], [g.ptr for g in db])
    torch.cuda.synchronize()
    for k, (g, w) in enumerate(zip(db, want)):
        assert g.guards_ok(), f"destination {k}: write outside the buffer"
        got = g.body().cpu().numpy().view(w.dtype).reshape(w.shape)
        if not np.array_equal(got, w):
            bad = np.argwhere(got != w)[:5]
            raise AssertionError(f"destination {k}: {int((got != w).sum())} elements differ, first at {bad.tolist()}")
    for g in sb:
        assert g.guards_ok()
    return p


@pytest.mark.gpu
@pytest.mark.parametrize("case", perm_cases(60, 78, big=True))
def test_gpu_permuted_against_oracle(case):
    shape, dt, sm, ss, sp, dm, ds, dp, kw = case
    print(f"permuted {case}", flush=True)
    _gpu_run(shape, dt, sm, ss, sp, dm, ds, dp, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", list(_NP))
@pytest.mark.parametrize("shape", [(130, 70), (128, 64), (33, 517), (5, 200, 3), (2, 40, 300), (4, 300, 257)])
def test_gpu_transpose_tiles(dt, shape):
    nd = len(shape)
    dp = tuple(range(nd - 2)) + (nd - 1, nd - 2)
    print(f"transpose tiles {dt} {shape}", flush=True)
    p = _gpu_run(shape, dt, (2,), "S^0" + "R" * (nd - 1), None, (2,), "R" * nd, dp)
    assert B.reshard_plan_transpose_chunks(p) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("fan", [1, 3])
@pytest.mark.parametrize("shape,es", TILE_EDGES)
def test_gpu_transpose_tile_edges(shape, es, fan):
    nd = len(shape)
    dp = tuple(range(nd - 2)) + (nd - 1, nd - 2)
    print(f"transpose tile edges {shape} es={es} fan={fan}", flush=True)
    p = _gpu_run(shape, _TILE_DT[es], (2,), "R" * (nd - 1) + "S^0", None, (fan, 2), "R" * (nd - 2) + "S^1R", dp)
    assert B.reshard_plan_transpose_chunks(p) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("fan", [1, 4])
@pytest.mark.parametrize("shape,es", TILE_LOOPS)
def test_gpu_transpose_chunks_of_many_tiles(shape, es, fan):
    print(f"transpose chunks of many tiles {shape} es={es} fan={fan}", flush=True)
    _gpu_run(shape, _TILE_DT[es], (1,), "RRR", None, (fan,), "RRR", (0, 2, 1), chunk_bytes=1 << 17)


@pytest.mark.gpu
@pytest.mark.parametrize("fan", [1, 2])
@pytest.mark.parametrize("shape,es,chunk", TILE_SETS)
def test_gpu_transpose_sets_of_tiles(shape, es, chunk, fan):
    print(f"transpose sets of tiles {shape} es={es} chunk={chunk} fan={fan}", flush=True)
    for kw in ({}, {"block_threads": 64}):
        _gpu_run(shape, _TILE_DT[es], (1,), "RRR", None, (fan,), "RRR", (0, 2, 1), chunk_bytes=chunk, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("shape,dt,sm,dm", HEADS)
def test_gpu_heads(shape, dt, sm, dm, back):
    print(f"heads {shape} {dt} {sm} {dm} back={back}", flush=True)
    heads_case(_gpu_run, shape, dt, sm, dm, back)


@pytest.mark.gpu
def test_gpu_transpose_unaligned_rows():
    for shape, dp in (((37, 90), (1, 0)), ((90, 37), (1, 0)), ((3, 37, 41), (2, 1, 0))):
        print(f"unaligned transpose {shape} {dp}", flush=True)
        _gpu_run(shape, "float16", (1,), "R" * len(shape), None, (2,), "S^0" + "R" * (len(shape) - 1), dp)


def _tunings(n, seed):
    rng = random.Random(seed)
    return [{k: v for k, v in (("chunk_bytes", rng.choice([0, 64, 1000, 8192, 40000])),
                               ("block_threads", rng.choice([0, 64, 128, 256, 512])),
                               ("max_wgs_per_cu", rng.choice([0, 2, 4, -1]))) if v} for _ in range(n)]


@pytest.mark.gpu
def test_gpu_permuted_soak():
    # 1,000 more permuted layouts under new seeds, each with its own chunk
    # size and then a random launch tuning, in one test
    for i, (case, tn) in enumerate(zip(perm_cases(1000, 5151, big=True), _tunings(1000, 5152))):
        shape, dt, sm, ss, sp, dm, ds, dp, kw = case
        for k in (kw, tn):
            print(f"permuted soak {i} {case} {k}", flush=True)
            _gpu_run(shape, dt, sm, ss, sp, dm, ds, dp, seed=i, **k)


@pytest.mark.gpu
@pytest.mark.parametrize("case,tuning", list(zip(perm_cases(120, 91), _tunings(120, 92))))
def test_gpu_permuted_fuzz_tunings(case, tuning):
    # seeded permuted layouts under random chunk sizes, workgroup sizes and
    # residency caps (the tile transpose, and the direct and gather chunks
    # of permuted plans, under every launch shape)
    shape, dt, sm, ss, sp, dm, ds, dp, _ = case
    print(f"permuted fuzz {case} {tuning}", flush=True)
    _gpu_run(shape, dt, sm, ss, sp, dm, ds, dp, **tuning)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["transposed2", "transposed5"])
def test_gpu_transposed_activation_full_size(name):
    # the GPT activations fp16 [8, 1024, 4096] (2,4) S^0 R S^1 -> (2,4)
    # R S^0 S^1 and fp16 [8, 2048, 12288] (4,8) R R S^{01} -> (4,8) R S^1 R
    # (4 replicas) with the destination in [batch, hidden, seq] order, in the
    # benchmark's launch configuration: every destination element compared
    # with the tensor transposed at the oracle's boxes, on the GPU
    import torch
    from paper_2211_05322_amd.workloads import make_tensor, workload_by_name
    w = workload_by_name(name)
    print(f"transposed activation {w.shape}", flush=True)
    x = make_tensor(w.shape, w.dtype, "normal", seed=0).cuda()
    n = len(w.shape)
    sc = B.reshard_plan(w.shape, w.dtype, (1,), "R" * n, w.src_mesh, w.src_spec, src_perm=None, dst_perm=w.src_perm)
    src = B.empty_shards(sc, 1)
    B.reshard_execute(sc, [x], src)
    p = B.reshard_plan(w.shape, w.dtype, w.src_mesh, w.src_spec, w.dst_mesh, w.dst_spec, src_perm=w.src_perm,
                       dst_perm=w.dst_perm)
    assert B.reshard_plan_transpose_chunks(p) > 0
    dst = B.empty_shards(p, 1)
    B.reshard_execute(p, src, dst)
    torch.cuda.synchronize()
    dims = oracle.parse_spec(w.dst_spec, n, len(w.dst_mesh))
    xb = x.view(torch.int16)
    for k, t in enumerate(dst):
        box = oracle.device_box(w.shape, w.dst_mesh, dims, k)
        ref = xb[tuple(slice(lo, hi) for lo, hi in box)].permute(*w.dst_perm)
        assert torch.equal(t.view(torch.int16), ref), f"destination {k}"


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dt,sp,dp", BIG_TRANSPOSES)
def test_gpu_transpose_above_4_gib(shape, dt, sp, dp):
    # every byte of a transposed buffer above 4 GiB against torch's permute
    import torch
    print(f"transpose above 4 GiB {shape} {dt} src_perm={sp} dst_perm={dp}", flush=True)
    bits = torch.uint8 if dt == "uint8" else torch.int16
    lo, hi = (0, 256) if dt == "uint8" else (-32768, 32768)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randint(lo, hi, shape, dtype=bits, device="cuda", generator=g)
    src = x.permute(*sp).contiguous() if sp else x
    p = B.reshard_plan(shape, dt, (1,), "RRR", (1,), "RRR", src_perm=sp, dst_perm=dp)
    dst = B.empty_shards(p, 1)
    assert dst[0].numel() * dst[0].element_size() > (4 << 30)
    B.reshard_execute(p, [src], dst)
    torch.cuda.synchronize()
    ref = x.permute(*dp) if dp else x
    assert torch.equal(dst[0].view(bits), ref)
