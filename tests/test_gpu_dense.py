"""GPU parity of large bf16 products whose operands are copied to dense aligned rows first (rows
that are not 16-byte aligned, many K-segments): against the fp64 oracle with the element bound of
test_gpu_parity, and bit for bit against the same product on the operands as they are (whether a call
takes the copies depends on where its operands lie and on free memory; its result must not).  Odd sizes,
column cuts inside 16-byte chunks, a share of K per replica of C, and operands in new places and
with new values under one plan (nothing of the copy may be kept)."""
import numpy as np
import pytest

import workloads
from oracle import matmul as omatmul
from tests.test_gpu_parity import _check, _check_bf16_out, _device_problem, _to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cyclic(M, K, N, nb, c):
    return dict(name=f"dense-bc{nb}-c{c}@{M}x{K}x{N}", M=M, K=K, N=N, dtype="bf16", nranks=8 * c,
                A=workloads.block_cyclic_desc(M, K, nb, nb, 2, 4, c), B=workloads.block_cyclic_desc(K, N, nb, nb, 2, 4, c),
                C=workloads.block_cyclic_desc(M, N, nb, nb, 2, 4, c), dist=("normal", 1.0), seeds=(61, 62))


def _uneven(M, K, N, s, b_cols=1):
    cuts = workloads.jittered_cuts
    return dict(name=f"dense-uneven@{M}x{K}x{N}", M=M, K=K, N=N, dtype="bf16", nranks=15,
                A=workloads.desc(M, K, cuts(M, 3, s), cuts(K, 5, s + 1), 3, 5),
                B=workloads.desc(K, N, cuts(K, 7, s + 2), cuts(N, b_cols, s + 5) if b_cols > 1 else [0, N], 7, b_cols),
                C=workloads.desc(M, N, cuts(M, 5, s + 3), cuts(N, 3, s + 4), 5, 3), dist=("uniform", 1.0), seeds=(63, 64))


CASES = [_cyclic(4101, 2051, 4099, 100, 1), _cyclic(3001, 4099, 4102, 99, 2), _uneven(8025, 2369, 4107, 77), _cyclic(4099, 3333, 4104, 100, 3),
         dict(_uneven(8025, 2369, 4107, 177, 2), stationary="B"),
         dict(_cyclic(4000, 4032, 8100, 100, 1), per_group=True)]     # (its merged macro-tiles would run in windows, cut along K)


def _on_the_operands(prob, cfg):
    """The same problem's plan on its own work list: merged macro-tiles where the plan has them (and not `per_group`)."""
    from paper_2510_08874_amd import binding
    flags = 0
    if prob.plan.num_merged_items() > 0 and not cfg.get("per_group"):
        plan = binding.Plan(cfg["A"], cfg["B"], cfg["C"], cfg["nranks"],
                            binding.STATIONARY_FLAGS[cfg.get("stationary", "C")] | binding.DMM_MERGE_ALWAYS)
    else:
        plan, flags = prob.plan, binding.DMM_NO_MERGE
    for t in prob.C.tensors:
        if t is not None:
            t.fill_(float("nan"))
    plan.execute_marshalled(prob.dtype_code, prob.args, flags | prob.c_flags, torch.cuda.current_stream().cuda_stream)
    assert not plan.ran_dense() and plan.small_tile() is None and not plan.ran_k_split()
    got = [prob.c_global(r) for r in range(cfg["C"]["replication"])]
    if plan is not prob.plan:
        plan.destroy()
    return got


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c["name"])
def test_products_on_dense_copies(cfg):
    A, B = workloads.make_operands(cfg)
    reps = cfg["C"]["replication"]
    prob = _device_problem(cfg, A, B, c_fill=float("nan"))
    prob.execute()
    assert prob.plan.ran_dense() and not prob.plan.ran_k_split()
    every = [prob.c_global(r) for r in range(reps)]
    got = every[0]
    A64, B64 = _to_f64(A, cfg), _to_f64(B, cfg)
    _check(got, omatmul.matmul(A, B, bf16=True), A64, B64, cfg, cfg["name"])
    for mine, own in zip(every, _on_the_operands(prob, cfg)):           # partial sums of the other replicas too
        assert np.array_equal(mine, own)
    prob.execute()                                       # the tables of the call before, the copy made anew
    assert np.array_equal(got, prob.c_global(0))
    for t in prob.A.tensors:                             # new values in the same place
        if t is not None:
            t.mul_(2.0)
    prob.execute()
    assert prob.plan.ran_dense()
    assert np.array_equal(2.0 * got, prob.c_global(0))   # (a power of two scales every sum exactly)
    moved = [None if t is None else t.clone() for t in prob.A.tensors]
    prob.A.tensors[:] = moved                            # the same values in new places
    prob.args = prob.plan.marshal(prob.A.tensors, prob.A.ld, prob.B.tensors, prob.B.ld, prob.C.tensors, prob.C.ld)
    prob.execute()
    assert np.array_equal(2.0 * got, prob.c_global(0))
    prob.close()


def test_bits_do_not_depend_on_where_the_operands_lie():
    """The same values in tiles at odd addresses, which the library copies, and in aligned ones, which it
    does not: the same bits."""
    M, K, N, block = 6656, 3840, 5376, workloads.block_desc
    cfg = dict(name="dense-or-not", M=M, K=K, N=N, dtype="bf16", nranks=64, A=block(M, K, 8, 8), B=block(K, N, 8, 8), C=block(M, N, 8, 8),
               dist=("normal", 1.0), seeds=(65, 66))
    A, B = workloads.make_operands(cfg)
    outs = []
    for odd in (True, False):
        prob = _device_problem(cfg, A, B, c_fill=float("nan"))
        if odd:                                          # the same tiles, two bytes further on
            for ts in (prob.A, prob.B):
                for i, t in enumerate(ts.tensors):
                    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
                    buf[1:].view(t.shape).copy_(t)
                    ts.tensors[i] = buf[1:].view(t.shape)
            prob.args = prob.plan.marshal(prob.A.tensors, prob.A.ld, prob.B.tensors, prob.B.ld, prob.C.tensors, prob.C.ld)
        prob.execute()
        outs.append((prob.c_global(0), prob.plan.ran_dense()))
        prob.close()
    assert [d for _, d in outs] == [True, False]
    assert np.array_equal(outs[0][0], outs[1][0])


def test_dense_copies_bf16_c_and_timing():
    """bf16 C tiles on the copies, bit for bit those on the operands; events around the kernels count the copy."""
    from paper_2510_08874_amd import binding
    cfg = CASES[2]
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, c_fill=float("nan"), c_dtype="bf16")
    prob.execute(flags=binding.DMM_TIMING)
    gemm_ms, reduce_ms = prob.plan.elapsed_ms()
    assert prob.plan.ran_dense() and 0.0 < gemm_ms < 100.0 and reduce_ms < 0.0
    got = prob.c_global(0)
    _check_bf16_out(got, omatmul.matmul(A, B, bf16=True), _to_f64(A, cfg), _to_f64(B, cfg), cfg["name"])
    assert np.array_equal(got, _on_the_operands(prob, cfg)[0])
    prob.execute()                                       # no events asked for: nothing to report
    assert prob.plan.elapsed_ms() == (-1.0, -1.0)
    prob.close()


def test_dense_copies_of_infinities_and_nan():
    """An infinity or a NaN in the operands reaches the elements it reaches on the operands as they are, and no others."""
    cfg = CASES[0]
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, c_fill=-1.0)
    prob.A.tensors[0][0, 99] = float("inf")              # the last column of a tile, in front of a filled-up step
    prob.A.tensors[2][3, 0] = float("nan")
    prob.B.tensors[5][99, 7] = float("-inf")
    prob.execute()
    assert prob.plan.ran_dense()
    got = prob.c_global(0)
    own = _on_the_operands(prob, cfg)[0]
    assert np.array_equal(got, own, equal_nan=True)
    assert 0 < np.count_nonzero(~np.isfinite(got)) <= 3 * 4102
    prob.close()


def test_plans_share_the_copies_buffers():
    """Kept plans of different sizes on copies, first on one stream, then each round on another of three: the
    buffers of the copies are shared, no call may see another's."""
    probs, wants = [], []
    for cfg in (CASES[0], CASES[1], CASES[2]):
        prob = _device_problem(cfg, *workloads.make_operands(cfg), c_fill=float("nan"))
        prob.execute()
        assert prob.plan.ran_dense()
        torch.cuda.synchronize()
        wants.append([None if t is None else t.clone() for t in prob.C.tensors])
        for t in prob.C.tensors:
            if t is not None:
                t.fill_(float("nan"))
        probs.append(prob)
    main, streams = torch.cuda.current_stream(), [torch.cuda.Stream() for _ in probs]
    for used in ([streams[0]] * 3, streams):
        for s in streams:
            s.wait_stream(main)
        for turn in range(6):
            for i, prob in enumerate(probs):
                s = used[(i + turn) % 3]
                s.wait_stream(used[(i + turn - 1) % 3])  # (of this problem's own last call: it wrote the same tiles of C)
                prob.execute(stream=s.cuda_stream)
                assert prob.plan.ran_dense()
        for s in streams:
            main.wait_stream(s)
        torch.cuda.synchronize()
        for prob, want in zip(probs, wants):
            for t, w in zip(prob.C.tensors, want):
                assert t is None or torch.equal(t, w)
    for prob in probs:
        prob.close()
