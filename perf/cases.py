"""The products this library is used for, as cases that can be timed and compared.

A case is a dict of plain values: what is called, the shape, the partitioning of the three
matrices, the element types.  `prepare` puts the tiles on the GPU, `run` is one pass through the
ABI binding, `work` is what a pass cannot do without, `tolerance` how far two correct
implementations may be apart.

  op         "execute": dmm_execute on a plan that is kept (the loop of a serving or training program)
             "plan_execute": dmm_plan + dmm_execute, a new plan every time (bench.py's step)
             "execute_broadcast": dmm_execute, then the summed replica 0 is copied to the other replicas
             "reduce": dmm_reduce_replicas alone
  layout     how A, B and C are cut and dealt to the ranks (`descriptors`)
  c          replicas of C (and of A and B in the "2d" layout)
  ld         leading dimensions are rounded up to a multiple of this many elements (1: packed)
"""
from __future__ import annotations

import math
from typing import Dict, List

import torch

import workloads
from paper_2510_08874_amd import binding

_DEFAULTS = dict(op="execute", layout="2d", ranks=8, c=1, dtype="bf16", c_dtype="f32", ld=1, nb=0, cut_seed=0, stationary="C",
                 dist="normal", scale=0.02)


def _case(**kw) -> Dict:
    return dict(_DEFAULTS, **kw)


def listed() -> List[Dict]:
    return [
        # the smallest call: latency of one launch on a plan that is kept
        _case(name="small_f32", layout="row_2d", ranks=4, m=256, k=256, n=256, dtype="f32", scale=1.0),
        # a small square product whose partitionings change from call to call: planning, table upload and launch count
        _case(name="square_2k_new_plan", op="plan_execute", layout="2d", ranks=4, m=2048, k=2048, n=2048, scale=1 / 64),
        # an ordinary product with misaligned row, column and 2-D blocks
        _case(name="misaligned_4k", layout="row_col", m=4096, k=4096, n=4096, scale=1 / 64),
        # a tensor-parallel linear layer on a long batch, activations stored in bf16 (the largest call)
        _case(name="tensor_parallel_prefill", layout="column", m=16384, k=8192, n=28672, c_dtype="bf16"),
        # the same kind of layer on a decode batch: a few rows against all of the weights
        _case(name="tensor_parallel_decode", layout="column", m=32, k=12288, n=49152, c_dtype="bf16"),
        # 2.5D: every matrix replicated twice over 32 ranks, partial sums of C added up; one new plan per step
        _case(name="replicated_25d_8k", op="plan_execute", layout="2d", ranks=32, c=2, m=8192, k=8192, n=8192, scale=8192 ** -0.5),
        # uneven cuts that match nowhere, odd sizes, packed rows
        _case(name="ragged_12k", layout="uneven", ranks=15, m=12289, k=9973, n=11003, cut_seed=5011, dist="uniform", scale=1.0),
        # single precision, odd sizes
        _case(name="ragged_f32_2k", layout="uneven", ranks=15, m=2501, k=1999, n=1777, dtype="f32", cut_seed=5011, dist="uniform", scale=1.0),
        # block-cyclic tiles much finer than the process grid; one new plan per step
        _case(name="block_cyclic_128", op="plan_execute", layout="cyclic", nb=128, m=8192, k=8192, n=8192, scale=8192 ** -0.5),
        # data-parallel weight gradient: every rank a partial sum of all of C, summed, then given to every rank
        _case(name="outer_product_all_reduce", op="execute_broadcast", layout="outer", ranks=8, c=8, m=4096, k=12288, n=4096),
        # a long inner dimension against a small result
        _case(name="long_inner", layout="row_col", m=1024, k=16384, n=1024),
        # the sum of partial results that other steps left in the replicas
        _case(name="replica_sum", op="reduce", layout="2d", ranks=64, c=4, m=8192, k=64, n=8192, scale=1.0),
    ]


def draw(rng) -> Dict:
    """One more case of the ranges above: sizes spread over their logarithm, most of them odd or ragged."""
    def size(lo, hi):
        x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        step = rng.choice((1, 1, 8, 64, 128))
        return max(lo, min(hi, (x + step - 1) // step * step))

    def most(case, flops):
        # a size is halved until the case costs no more than `flops`
        while 2.0 * case["m"] * case["k"] * case["n"] > flops:
            big = max(("m", "k", "n"), key=lambda d: case[d])
            case[big] = case[big] // 2
        return case

    ld, new = rng.choice((1, 8)), rng.choice(("execute", "plan_execute"))
    kind = rng.choice(("small", "square", "layer", "layer", "replicated", "uneven", "f32", "cyclic", "outer", "long", "reduce"))
    if kind == "small":
        return _case(op=new, layout=rng.choice(("row_2d", "row_col", "2d")), ranks=rng.choice((4, 8)), m=size(64, 1024), k=size(64, 1024),
                     n=size(64, 1024), dtype=rng.choice(("bf16", "f32")), ld=ld, scale=1.0)
    if kind == "square":
        return _case(op=new, layout=rng.choice(("2d", "row_col")), ranks=rng.choice((4, 8, 16)), m=size(1024, 6144), k=size(1024, 6144),
                     n=size(1024, 6144), ld=ld, stationary=rng.choice("CBA"))
    if kind == "layer":
        return most(_case(layout="column", m=size(1, 16384), k=size(2048, 16384), n=size(4096, 49152), c_dtype=rng.choice(("bf16", "f32")), ld=8), 6e12)
    if kind == "replicated":
        return _case(op=new, layout="2d", ranks=rng.choice((8, 32)), c=2, m=size(1024, 8192), k=size(1024, 8192), n=size(1024, 8192), ld=ld)
    if kind == "uneven":
        return _case(layout="uneven", ranks=15, m=size(1024, 12288), k=size(1024, 10240), n=size(1024, 11008), ld=ld,
                     cut_seed=rng.randrange(1, 10000), dist="uniform", scale=1.0)
    if kind == "f32":
        return most(_case(op=new, layout=rng.choice(("2d", "row_col", "uneven")), ranks=16, m=size(512, 6144), k=size(512, 6144), n=size(512, 6144),
                          dtype="f32", ld=ld, cut_seed=rng.randrange(1, 10000)), 3e11)
    if kind == "cyclic":
        return _case(op=new, layout="cyclic", nb=rng.choice((64, 100, 128, 256)), m=size(1024, 8192), k=size(1024, 8192), n=size(1024, 8192), ld=ld)
    if kind == "outer":
        c = rng.choice((2, 4, 8))
        return _case(op=rng.choice(("execute", "execute_broadcast")), layout="outer", ranks=c, c=c, m=size(1024, 8192), k=size(2048, 16384),
                     n=size(1024, 8192), ld=ld)
    if kind == "long":
        return _case(layout=rng.choice(("row_col", "2d", "cyclic")), nb=128, m=size(128, 1536), k=size(8192, 49152), n=size(128, 1536),
                     dtype=rng.choice(("bf16", "bf16", "f32")), ld=ld)
    c = rng.choice((2, 3, 4, 8))
    return _case(op="reduce", layout="2d", ranks=c * 4, c=c, m=size(512, 8192), k=64, n=size(512, 8192), ld=ld, scale=1.0)


# ---- partitionings ---------------------------------------------------------------------------------

def _grid(p):
    """p ranks as a process grid, as square as p allows, more rows than columns."""
    q = max(d for d in range(1, int(p ** 0.5) + 1) if p % d == 0)
    return p // q, q


def descriptors(case):
    m, k, n, p, c, layout = (case[x] for x in ("m", "k", "n", "ranks", "c", "layout"))
    block = workloads.block_desc
    if layout == "row_2d":        # row blocks times 2-D blocks
        r, q = _grid(p)
        return block(m, k, p, 1), block(k, n, r, q), block(m, n, r, q)
    if layout == "row_col":       # row blocks times column blocks, C in 2-D blocks
        r, q = _grid(p)
        return block(m, k, p, 1), block(k, n, 1, p), block(m, n, r, q)
    if layout == "2d":            # 2-D blocks, all three matrices replicated c times (2.5D)
        r, q = _grid(p // c)
        return block(m, k, r, q, replication=c), block(k, n, r, q, replication=c), block(m, n, r, q, replication=c)
    if layout == "column":        # A on every rank, B and C in column blocks
        return block(m, k, 1, 1, replication=p), block(k, n, 1, p), block(m, n, 1, p)
    if layout == "outer":         # column blocks times row blocks, a partial sum of C on every rank
        return block(m, k, 1, p), block(k, n, p, 1), block(m, n, 1, 1, replication=p)
    if layout == "uneven":        # 3 x 5, 7 x 1 and 5 x 3 uneven blocks
        s, cuts = case["cut_seed"], workloads.jittered_cuts
        return (workloads.desc(m, k, cuts(m, 3, s), cuts(k, 5, s + 1), 3, 5), workloads.desc(k, n, cuts(k, 7, s + 2), [0, n], 7, 1),
                workloads.desc(m, n, cuts(m, 5, s + 3), cuts(n, 3, s + 4), 5, 3))
    if layout == "cyclic":        # nb x nb tiles dealt to the process grid
        nb, (q, r) = case["nb"], _grid(p)
        cyclic = workloads.block_cyclic_desc
        return cyclic(m, k, nb, nb, r, q), cyclic(k, n, nb, nb, r, q), cyclic(m, n, nb, nb, r, q)
    raise KeyError(layout)


class _Tiles:
    """The tiles of one matrix: per replica one buffer (a rank's memory pool) that holds them one
    after another, each at a multiple of 512 bytes, as an allocator would place them."""

    def __init__(self, desc, dtype, ld_multiple):
        rc, cc = desc["row_cuts"], desc["col_cuts"]
        size = 2 if dtype == torch.bfloat16 else 4
        offsets, self.ld, total = [], [], 0
        for r0, r1 in zip(rc, rc[1:]):
            for c0, c1 in zip(cc, cc[1:]):
                ld = max(-(-(c1 - c0) // ld_multiple) * ld_multiple, 1)
                offsets.append(total if r1 > r0 and c1 > c0 else None)
                self.ld.append(ld)
                total += -(-(r1 - r0) * ld * size // 512) * 512 // size
        self.ld *= desc["replication"]
        self.buffers = [torch.zeros(total, dtype=dtype, device="cuda") for _ in range(desc["replication"])]
        self.pointers = [None if o is None else b.data_ptr() + o * size for b in self.buffers for o in offsets]

    def fill(self, case, generator, copies):
        """Values of the case's distribution; `copies`: all replicas hold the same ones."""
        for i, b in enumerate(self.buffers):
            if i and copies:
                b.copy_(self.buffers[0])
            elif case["dist"] == "normal":
                b.normal_(0.0, case["scale"], generator=generator)
            else:
                b.uniform_(-case["scale"], case["scale"], generator=generator)


# ---- one pass --------------------------------------------------------------------------------------

def prepare(case, seed):
    """The tiles on the GPU, the plan that a program keeps, the marshalled argument tables."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    da, db, dc = descriptors(case)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    C = _Tiles(dc, torch.bfloat16 if case["c_dtype"] == "bf16" else torch.float32, case["ld"])
    flags = binding.STATIONARY_FLAGS[case["stationary"]]
    state = dict(op=case["op"], descs=(da, db, dc), ranks=case["ranks"], plan_flags=flags, C=C,
                 plan=binding.Plan(da, db, dc, case["ranks"], flags), in_flight=[],
                 dtype=binding.DMM_BF16 if case["dtype"] == "bf16" else binding.DMM_F32,
                 flags=binding.DMM_C_BF16 if case["c_dtype"] == "bf16" else 0, stream=torch.cuda.current_stream().cuda_stream)
    if case["op"] == "reduce":
        C.fill(case, gen, copies=False)
        return state
    A, B = _Tiles(da, dtype, case["ld"]), _Tiles(db, dtype, case["ld"])
    A.fill(case, gen, copies=True)
    B.fill(case, gen, copies=True)
    state.update(A=A, B=B, args=state["plan"].marshal(A.pointers, A.ld, B.pointers, B.ld, C.pointers, C.ld))
    return state


def run(state):
    """One pass; the whole of every replica of C."""
    op, plan, C = state["op"], state["plan"], state["C"]
    if op == "reduce":
        plan.reduce_replicas(C.pointers, C.ld, 0, state["stream"])
    elif op == "plan_execute":
        # the plans of the last three steps are kept, the one before them has long finished
        plan = binding.Plan(*state["descs"], state["ranks"], state["plan_flags"])
        plan.execute_marshalled(state["dtype"], state["args"], state["flags"], state["stream"])
        state["in_flight"].append(plan)
        if len(state["in_flight"]) > 3:
            state["in_flight"].pop(0).destroy()
    else:
        plan.execute_marshalled(state["dtype"], state["args"], state["flags"], state["stream"])
        if op == "execute_broadcast":
            plan.broadcast_replica(C.pointers, C.ld, 0, state["stream"])
    return C.buffers


def work(case):
    m, k, n, c = case["m"], case["k"], case["n"], case["c"]
    if case["op"] == "reduce":
        return {"bytes": (c + 1) * 4.0 * m * n, "flops": (c - 1) * 1.0 * m * n}
    es, c_es = (2 if case[t] == "bf16" else 4 for t in ("dtype", "c_dtype"))
    return {"bytes": float(es) * (m * k + k * n) + float(c_es) * c * m * n, "flops": 2.0 * m * k * n}


def tolerance(case):
    # about four times what the listed and drawn cases show against the product in 64 bits; two
    # correct orders of the fp32 sums differ by as much
    if case["op"] == "reduce":
        return "exact"                            # one addition per replica in a stated order
    if case["c_dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}       # one rounding to bf16: 1.66e-3 and half an ulp, 3.9e-3
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}         # 7.7e-7 and 7.1e-6 at k = 1856, growing with the root of k (largest: 49152)
    return {"rel": 4e-6, "max": 4e-5}             # products of bf16 are exact: 5.7e-7 and 5.6e-6
