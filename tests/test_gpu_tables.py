"""Small work tables travel with a kernel on the caller's stream, and a call's last launch records the event that
stands for it: calls of one plan on two streams, with buffers that change from call to call, are each right, one
after another and with all of them enqueued before the first has begun."""
import numpy as np
import pytest

import workloads
from paper_2510_08874_amd import binding
from paper_2510_08874_amd.tiles import DeviceProblem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dims", [("bf16", (300, 520, 260)), ("f32", (130, 260, 140)), ("bf16", (300, 20000, 260))])
def test_buffers_change_on_two_streams(dtype, dims):
    M, K, N = dims
    block = workloads.block_desc
    probs = []
    for seed in (3, 4, 5):
        cfg = dict(name="tables", M=M, K=K, N=N, nranks=4, dtype=dtype, A=block(M, K, 2, 2), B=block(K, N, 2, 2), C=block(M, N, 2, 2),
                   dist=("normal", 1.0), seeds=(seed, seed + 10))
        A, B = workloads.make_operands(cfg)
        p = DeviceProblem(cfg, A, B, c_fill=float("nan"))
        probs.append(p)
    want = []
    for p in probs:
        p.execute()
        torch.cuda.synchronize()
        want.append(p.c_global(0))
        assert np.isfinite(want[-1]).all()
    plan = probs[0].plan
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for r in range(12):
        i, s = r % 3, streams[(r // 2) % 2]
        p = probs[i]
        for t in p.C.tensors:
            if t is not None:
                t.fill_(float("nan"))
        torch.cuda.synchronize()
        args = plan.marshal(p.A.tensors, p.A.ld, p.B.tensors, p.B.ld, p.C.tensors, p.C.ld)
        code = binding.DMM_BF16 if dtype == "bf16" else binding.DMM_F32
        for _ in range(2):                       # (the second call finds its table in place)
            plan.execute_marshalled(code, args, 0, s.cuda_stream)
        s.synchronize()
        assert np.array_equal(p.c_global(0), want[i]), (r, i)
    for p in probs:
        p.close()


# (cuts: tiles a side of A and B, and of C; alternate: every other call runs the macro-tiles, whose table is copied)
@pytest.mark.parametrize("dtype,dims,cuts,alternate,runs", [
    ("bf16", (300, 250, 260), (2, 2), False, False),
    ("f32", (130, 100, 140), (2, 2), False, False),
    ("bf16", (300, 20000, 260), (2, 2), False, True),     # partial tiles in a buffer that all calls share
    ("bf16", (700, 900, 600), (3, 6), True, True),        # ... a table of 2232 bytes, written, and one of 8064, copied
])
def test_calls_that_overlap_on_two_streams(dtype, dims, cuts, alternate, runs):
    """A few milliseconds of other work lie ahead on both streams while the calls are enqueued, none of them waited for."""
    M, K, N = dims
    block, (n, nc) = workloads.block_desc, cuts
    probs, want = [], {}
    for seed in (3, 4, 5):
        cfg = dict(name="tables", M=M, K=K, N=N, nranks=36, dtype=dtype, A=block(M, K, n, n), B=block(K, N, n, n), C=block(M, N, nc, nc),
                   dist=("normal", 1.0), seeds=(seed, seed + 10))
        p = DeviceProblem(cfg, *workloads.make_operands(cfg), c_fill=float("nan"))
        for flags in (0, binding.DMM_NO_MERGE) if alternate else (0,):
            p.execute(flags=flags)
            torch.cuda.synchronize()
            assert (p.plan.small_tile() is None) == (flags != 0) and (flags or (p.plan.last_kernels().small_runs > 1) == runs)
            want[len(probs), flags] = p.c_global(0)
            assert np.isfinite(want[len(probs), flags]).all()
        probs.append(p)
    plan, streams = probs[0].plan, [torch.cuda.Stream(), torch.cuda.Stream()]
    code = binding.DMM_BF16 if dtype == "bf16" else binding.DMM_F32
    calls = []
    for r in range(24):
        i, flags = r % 3, binding.DMM_NO_MERGE if alternate and r % 2 else 0
        C = [torch.full_like(t, float("nan")) for t in probs[i].C.tensors]
        calls.append((i, flags, streams[(r // 2) % 2 if r < 12 else r % 2], C,
                      plan.marshal(probs[i].A.tensors, probs[i].A.ld, probs[i].B.tensors, probs[i].B.ld, C, probs[i].C.ld)))
    x = torch.randn(4096, 4096, device="cuda").to(torch.bfloat16)
    torch.cuda.synchronize()
    ahead = []
    for s in streams:
        with torch.cuda.stream(s):
            ahead += [torch.mm(x, x) for _ in range(16)]
    for i, flags, s, _, args in calls:
        plan.execute_marshalled(code, args, flags, s.cuda_stream)
    torch.cuda.synchronize()
    for r, (i, flags, _, C, _) in enumerate(calls):
        kept, probs[i].C.tensors = probs[i].C.tensors, C
        got = probs[i].c_global(0)
        probs[i].C.tensors = kept
        assert np.array_equal(got, want[i, flags]), (r, i, flags)
    for p in probs:
        p.close()
