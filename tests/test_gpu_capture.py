"""A plan's calls under HIP graph capture, after the plan has run on the stream that is captured: macro-tiles
on the operands, dense copies, tiles cut along K.  Every replay, with eager work in between, gives
bit for bit what the eager call gave."""
import pytest

import workloads
from tests.test_gpu_parity import _device_problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _row_col(M, K, N, dtype="bf16"):
    block = workloads.block_desc
    return dict(name=f"capture-{dtype}-{M}x{K}x{N}", M=M, K=K, N=N, dtype=dtype, nranks=8, A=block(M, K, 8, 1), B=block(K, N, 1, 8),
                C=block(M, N, 4, 2), dist=("normal", 1.0), seeds=(71, 72))


def _cyclic(M, K, N, nb):
    cyclic = workloads.block_cyclic_desc
    return dict(name=f"capture-bc{nb}-{M}x{K}x{N}", M=M, K=K, N=N, dtype="bf16", nranks=8, A=cyclic(M, K, nb, nb, 2, 4, 1),
                B=cyclic(K, N, nb, nb, 2, 4, 1), C=cyclic(M, N, nb, nb, 2, 4, 1), dist=("normal", 1.0), seeds=(73, 74))


@pytest.mark.parametrize("cfg,dense,small,split", [
    (_row_col(4096, 1024, 4096), False, False, False),
    (_cyclic(4101, 2051, 4099, 100), True, False, False),
    (_row_col(1024, 8192, 1024), False, True, True),
    (_row_col(256, 256, 256, "f32"), False, True, True),
], ids=lambda x: x["name"] if isinstance(x, dict) else "")
def test_calls_under_capture(cfg, dense, small, split):
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, c_fill=float("nan"))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    for _ in range(2):
        prob.execute(stream=stream.cuda_stream)
    torch.cuda.synchronize()
    assert (prob.plan.ran_dense(), prob.plan.small_tile() is not None, prob.plan.ran_k_split()) == (dense, small, split)
    tiles = [t for t in prob.C.tensors if t is not None]
    want = [t.clone() for t in tiles]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        prob.execute(stream=stream.cuda_stream)
    for _ in range(3):
        for t in tiles:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(tiles, want))
        prob.execute()                                       # eager work on another stream
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(tiles, want))
    del graph
    prob.close()
