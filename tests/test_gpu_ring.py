"""GPU parity of the ring kernels (bf16 tiles of 32, 64 and 128 x 128, operands straight into a ring of LDS
stages) where their loop changes form: fewer steps than stages, K tails of every kind (whole chunks, parts of a
chunk, segments shorter than one), rows shorter than a chunk, column edges at the end of a tile buffer, more
segments than their descriptor area holds.  Each against the fp64 oracle (element bound of test_gpu_parity) and,
where K is not cut, bit for bit against the macro-tile kernels; the padding holds infinities."""
import numpy as np
import pytest

import workloads
from oracle import matmul as omatmul
from tests.test_gpu_parity import _check, _device_problem, _to_f64
from tests.test_gpu_small import _pad_with_inf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cuts(total, step):
    return list(range(0, total, step)) + [total]


def _problem(M, K, N, ak, bk, mcut, ncut):
    """A in column strips of ak, B in row strips of bk, C in tiles of mcut x ncut."""
    da, db, dc = _cuts(K, ak), _cuts(K, bk), (_cuts(M, mcut), _cuts(N, ncut))
    A = workloads.desc(M, K, [0, M], da, 1, len(da) - 1)
    B = workloads.desc(K, N, db, [0, N], len(db) - 1, 1)
    C = workloads.desc(M, N, dc[0], dc[1], len(dc[0]) - 1, len(dc[1]) - 1)
    ranks = max(len(da) - 1, len(db) - 1, (len(dc[0]) - 1) * (len(dc[1]) - 1))
    return dict(name=f"ring-{M}x{K}x{N}-{ak}-{bk}", M=M, K=K, N=N, nranks=ranks, dtype="bf16", A=A, B=B, C=C, dist=("normal", 1.0), seeds=(17, 18))


@pytest.mark.parametrize("ldm", [1, 8])
@pytest.mark.parametrize("M,K,N,ak,bk,mcut,ncut", [
    (128, 64, 128, 64, 64, 128, 128),       # one step
    (130, 129, 131, 129, 129, 130, 131),    # three steps, the last of one element
    (31, 195, 127, 195, 65, 31, 127),       # four, tails of one
    (300, 324, 520, 67, 110, 300, 520),     # tails of three and more in all segments
    (64, 250, 1000, 5, 250, 64, 1000),      # segments shorter than a chunk
    (257, 320, 384, 56, 320, 100, 72),      # whole chunks missing; tiles across C's cuts
    (40, 700, 3, 350, 700, 40, 3),          # rows of B of six bytes
    (33, 200, 12, 200, 77, 33, 12),         # chunks of B past the end of its buffers in every segment
    (1400, 1290, 1500, 129, 1290, 1400, 1500),   # 128 x 128 tiles, K tails, uncut
    (1300, 6000, 150, 24, 40, 65, 150),     # several hundred segments: descriptors in windows
    (1290, 4000, 1290, 18, 4000, 10, 1290), # ... and many row pieces
])
def test_ring(M, K, N, ak, bk, mcut, ncut, ldm):
    from paper_2510_08874_amd import binding
    cfg = _problem(M, K, N, ak, bk, mcut, ncut)
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, ld_multiple=ldm, c_fill=float("nan"))
    _pad_with_inf(prob)
    prob.execute()
    assert prob.plan.small_tile() is not None
    split = prob.plan.ran_k_split()
    got = prob.c_global(0)
    _check(got, omatmul.matmul(A, B, bf16=True), _to_f64(A, cfg), _to_f64(B, cfg), cfg, cfg["name"])
    if not split:
        prob.execute(flags=binding.DMM_NO_MERGE)
        if not prob.plan.ran_k_split():
            assert np.array_equal(got, prob.c_global(0))
    prob.close()
