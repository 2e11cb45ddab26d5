"""Small work tables travel with a kernel on the caller's stream, and a call's last launch records the event that
stands for it: calls of one plan on two streams, with buffers that change from call to call, are each right."""
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
