"""The reshards whose speed is measured, as a training or serving program issues them.

One case is one resharding task: a tensor, the mesh and sharding spec it is
laid out under, those it is wanted under, and each side's buffer order.  A
program plans the task once and executes it every iteration; `prepare` makes
the plan, the source shards and the receivers' buffers, and `run` executes.
Every result is a copy of bits, so outputs are compared exactly.
"""

import math

import torch

from paper_2211_05322_amd import binding as B

DTYPES = {"float16": 2, "bfloat16": 2, "float32": 4, "uint8": 1, "int64": 8}


def _case(name, dtype, shape, src_mesh, src_spec, dst_mesh, dst_spec, src_perm="", dst_perm=""):
    return {"name": name, "dtype": dtype, "shape": shape, "src_mesh": src_mesh, "src_spec": src_spec,
            "dst_mesh": dst_mesh, "dst_spec": dst_spec, "src_perm": src_perm, "dst_perm": dst_perm}


def listed():
    return [
        # a small fp32 tensor, columns to rows, two replicas: call and launch latency
        _case("small_fp32_cols_to_rows", "float32", "256,1024", "1,2", "S^1 R", "2,2", "R S^0"),
        # one decode step of a 64-sequence batch, hidden shards to every device
        _case("decode_fp16_to_8rep", "float16", "64,1,5120", "2,4", "R R S^{01}", "2,4", "R R R"),
        # GPT layer activation between pipeline stages, batch shards to sequence shards
        _case("gpt_act_fp16_batch_to_seq", "float16", "8,1024,4096", "2,4", "S^0 R S^1", "2,4", "R S^0 S^1"),
        # hidden shards gathered onto 8 replicas: the largest
        _case("act_fp16_hidden_to_8rep", "float16", "16,2048,5120", "2,4", "R R S^{01}", "2,4", "R R R"),
        # U-Transformer skip connection, its height (66) split unevenly in four, two replicas
        _case("utrans_skip_fp16_uneven_h", "float16", "32,512,66,64", "2,2", "S^0 S^1 R R", "4,2", "R R S^0 R"),
        # GPT-3-width activation, 32 hidden shards to 8 sequence shards on 4 replicas (forward)
        _case("gpt3_act_fp16_to_seq_4rep", "float16", "8,2048,12288", "4,8", "R R S^{01}", "4,8", "R S^1 R"),
        # its gradient on the way back: sequence shards to 32 hidden shards (backward)
        _case("gpt3_grad_bf16_seq_to_hidden", "bfloat16", "8,2048,12288", "4,8", "R S^1 R", "4,8", "R R S^{01}"),
        # a width the shard count does not divide: misaligned segments, 4 replicas
        _case("uneven_act_fp16_to_4rep", "float16", "8,2048,12300", "4,8", "R R S^{01}", "4,8", "R S^1 R"),
        # the receivers keep the activation [batch, hidden, seq]: a transpose, 4 replicas
        _case("transposed_act_fp16_4rep", "float16", "8,2048,12288", "4,8", "R R S^{01}", "4,8", "R S^1 R",
              "", "0,2,1"),
        # the same change of order on ragged extents (a next-token batch of 2047, an odd width)
        _case("transposed_act_bf16_ragged", "bfloat16", "8,2047,4098", "2,4", "S^0 R S^1", "2,4", "R S^0 S^1",
              "", "0,2,1"),
        # attention heads: [batch, seq, head, dim] to [batch, head, seq, dim], sequence shards to head shards
        _case("heads_bf16_seq_to_head", "bfloat16", "8,2048,32,128", "2,4", "R S^{01} R R", "2,4", "R R S^1 R",
              "", "0,2,1,3"),
        # byte tensor with odd rows (a mask), row shards to column shards, two replicas
        _case("mask_u8_odd_rows_to_cols", "uint8", "64,1025,1001", "2,4", "R S^{01} R", "4,2", "R R S^0"),
    ]


# ------------------------------------------------------------------ the ranges

# (shapes' rank, source mesh, source spec, destination mesh, destination spec): layouts of activations,
# gradients, weights and feature maps between two stages, fan-outs 1 to 32
_LAYOUTS = {
    3: [("2,4", "S^0 R S^1", "2,4", "R S^0 S^1"), ("2,4", "R R S^{01}", "2,4", "R R R"),
        ("4,8", "R R S^{01}", "4,8", "R S^1 R"), ("4,8", "R S^1 R", "4,8", "R R S^{01}"),
        ("2,4", "S^0 R R", "2,4", "S^0 R S^1"), ("2,4", "R S^{01} R", "4,2", "R R S^0"),
        ("2,4", "R S^0 R", "2,4", "S^0 R R"), ("1,4", "S^1 R R", "2,4", "R R R"),
        ("2,4", "R S^0 R", "2,4", "R R S^0"), ("2,4", "S^0 R R", "3,4", "S^0 R R"),
        ("1", "R R R", "4,8", "R R R")],
    2: [("1,2", "S^1 R", "2,2", "R S^0"), ("2,4", "S^0 S^1", "2,4", "S^1 S^0"),
        ("1,8", "R S^1", "2,4", "R R"), ("2,2", "S^{01} R", "4,2", "R S^0")],
    4: [("2,2", "S^0 S^1 R R", "4,2", "R R S^0 R"), ("2,4", "R S^{01} R R", "2,4", "R R S^1 R"),
        ("2,4", "S^0 R S^1 R", "2,4", "S^0 S^1 R R")],
}
_PERMS = {3: ["", "", "", "0,2,1", "1,0,2"], 2: ["", "", "1,0"], 4: ["", "", "0,2,1,3", "0,2,3,1"]}
_MIN_BYTES, _MAX_BYTES = 64 << 10, 2 << 30  # read + written


def draw(rng):
    while True:
        rank = rng.choice([2, 3, 3, 3, 4])
        src_mesh, src_spec, dst_mesh, dst_spec = rng.choice(_LAYOUTS[rank])
        dtype = rng.choice(["float16", "bfloat16", "float16", "bfloat16", "float32", "uint8", "int64"])
        src_perm, dst_perm = "", rng.choice(_PERMS[rank])
        if dst_perm and rng.random() < 0.3:  # the way back of a permuted layout
            src_perm, dst_perm = dst_perm, ""
        total = math.exp(rng.uniform(math.log(_MIN_BYTES), math.log(_MAX_BYTES)))
        # leading extents log-uniform over what activations and feature maps have, the last from the size
        if rank == 2:
            shape = [int(2 ** rng.uniform(5, 13))]
        elif rank == 3:
            shape = [int(2 ** rng.uniform(2, 6)), int(2 ** rng.uniform(5, 11.5))]
        else:
            shape = [int(2 ** rng.uniform(2, 5)), int(2 ** rng.uniform(5, 11)), int(2 ** rng.uniform(4, 6.5))]
        case = _case("", dtype, "", src_mesh, src_spec, dst_mesh, dst_spec, src_perm, dst_perm)
        probe = dict(case, shape=",".join(map(str, shape + [840])))
        per = work(probe)["bytes"] / 840.0  # bytes per unit of the last extent
        shape.append(int(total / per))
        if not 24 <= shape[-1] <= 32768:
            continue
        if rng.random() < 0.5:  # widths that shards and vectors divide; the others stay as drawn, odd ones among them
            shape = [shape[0]] + [max(16, s // 16 * 16) for s in shape[1:-1]] + [max(64, shape[-1] // 64 * 64)]
        case["shape"] = ",".join(map(str, shape))
        del case["name"]
        if work(case)["bytes"] <= _MAX_BYTES:
            return case


# ------------------------------------------------------------------ a case's layouts

def _ints(text):
    return [int(x) for x in text.split(",")] if text else []


def _axes(spec):
    """Mesh axes of each tensor dimension of "R S^0 S^{01}" (major to minor)."""
    return [[int(c) for c in tok if c.isdigit()] for tok in spec.split()]


def _boxes(shape, mesh, spec):
    """Per device (row-major), the slices of the tensor it holds: balanced splits, the first shards one longer."""
    n = math.prod(mesh)
    boxes = []
    for dev in range(n):
        coord, r = [], dev
        for m in reversed(mesh):
            coord.insert(0, r % m)
            r //= m
        box = []
        for length, axes in zip(shape, _axes(spec)):
            k, j = 1, 0
            for a in axes:
                k, j = k * mesh[a], j * mesh[a] + coord[a]
            q, rem = divmod(length, k)
            lo = j * q + min(j, rem)
            box.append((lo, lo + q + (1 if j < rem else 0)))
        boxes.append(box)
    return boxes


def _shards(t, mesh, spec, perm):
    """Each device's buffer: its slice, dimensions in the buffer's order, dense."""
    out = []
    for box in _boxes(t.shape, mesh, spec):
        s = t[tuple(slice(lo, hi) for lo, hi in box)]
        # a buffer of its own, also where the slice is already dense
        out.append((s.permute(perm) if perm else s).clone(memory_format=torch.contiguous_format))
    return out


def _tensor(case, seed):
    """The logical tensor: activations and gradients N(0,1), byte masks and token ids whole numbers."""
    shape, dtype = _ints(case["shape"]), getattr(torch, case["dtype"])
    g = torch.Generator(device="cuda").manual_seed(seed)
    if dtype == torch.uint8:
        return torch.randint(0, 256, shape, generator=g, device="cuda", dtype=dtype)
    if dtype == torch.int64:
        return torch.randint(0, 1 << 40, shape, generator=g, device="cuda", dtype=dtype)
    if dtype == torch.float32:
        return torch.randn(shape, generator=g, device="cuda")
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


# ------------------------------------------------------------------ prepare, run, compare

def prepare(case, seed):
    perms = [tuple(_ints(case[k])) or None for k in ("src_perm", "dst_perm")]
    plan = B.reshard_plan(_ints(case["shape"]), case["dtype"], _ints(case["src_mesh"]), case["src_spec"],
                          _ints(case["dst_mesh"]), case["dst_spec"], src_perm=perms[0], dst_perm=perms[1])
    B.reshard_plan_upload(plan)
    src = _shards(_tensor(case, seed), _ints(case["src_mesh"]), case["src_spec"], perms[0])
    dst = B.empty_shards(plan, 1)
    return {"plan": plan, "src": src, "dst": dst, "src_ptrs": B.pointer_array(src), "dst_ptrs": B.pointer_array(dst)}


def run(state):
    B.reshard_execute(state["plan"], state["src_ptrs"], state["dst_ptrs"])
    return state["dst"]


def work(case):
    """Every element read once, every receiver's shard written once; no arithmetic."""
    shape, es = _ints(case["shape"]), DTYPES[case["dtype"]]
    written = sum(math.prod(hi - lo for lo, hi in box)
                  for box in _boxes(shape, _ints(case["dst_mesh"]), case["dst_spec"]))
    return {"bytes": es * (math.prod(shape) + written), "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The receivers' shards cut straight from the logical tensor."""
    return _shards(_tensor(case, seed), _ints(case["dst_mesh"]), case["dst_spec"], tuple(_ints(case["dst_perm"])) or None)
