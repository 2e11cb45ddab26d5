"""GPU parity of the kernels for small and skinny products (tiles of 32 to 128 rows and columns
cut across the cuts of A, B and C): against the fp64 oracle with the element bound of
test_gpu_parity, and bitwise against the macro-tile kernels (DMM_NO_MERGE) where the tiles are not
cut along K (every shape but 32 x 32, whose waves share K).  Every case names the shape that has to run.  The padding of every operand row holds infinities: a read past a segment that
reached a sum would show as NaN."""
import numpy as np
import pytest

import workloads
from oracle import matmul as omatmul
from tests.test_gpu_parity import _check, _device_problem, _to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cfg(dims, dtype, kind, seed=5):
    M, K, N = dims
    if kind == "whole":
        d = [workloads.block_desc(r, c, 1, 1) for r, c in ((M, K), (K, N), (M, N))]
        p = 1
    elif kind == "blocks":              # row blocks x column blocks, C in 2-D blocks
        d = [workloads.block_desc(M, K, 8, 1), workloads.block_desc(K, N, 1, 8), workloads.block_desc(M, N, 4, 2)]
        p = 8
    elif kind == "column":              # A on every rank, B and C in column blocks
        d = [workloads.block_desc(M, K, 1, 1, replication=4), workloads.block_desc(K, N, 1, 4), workloads.block_desc(M, N, 1, 4)]
        p = 4
    else:                               # uneven cuts that match nowhere
        cuts = workloads.jittered_cuts
        d = [workloads.desc(M, K, cuts(M, 3, seed), cuts(K, 5, seed + 1), 3, 5), workloads.desc(K, N, cuts(K, 7, seed + 2), [0, N], 7, 1),
             workloads.desc(M, N, cuts(M, 5, seed + 3), cuts(N, 3, seed + 4), 5, 3)]
        p = 15
    return dict(name=f"small-{kind}-{dtype}-{M}x{K}x{N}", M=M, K=K, N=N, nranks=p, dtype=dtype, A=d[0], B=d[1], C=d[2],
                dist=("normal", 1.0), seeds=(91, 92))


def _pad_with_inf(prob):
    for ts in (prob.A, prob.B):
        cells = [(i, j) for _ in range(len(ts.tensors) // (ts.gr * ts.gc)) for i in range(ts.gr) for j in range(ts.gc)]
        for t, (ti, tj) in zip(ts.tensors, cells):
            if t is not None:
                _, _, c0, c1 = ts.bounds(ti, tj)
                t[:, c1 - c0:] = float("inf")


S, H, B, T, F = (32, 128), (64, 128), (128, 128), (32, 32), (64, 64)      # the tiles: three for bf16, two for fp32


# (tile: that of the shape that has to run; runs: K is cut into several ranges)
@pytest.mark.parametrize("dims,dtype,kind,ldm,tile,runs", [
    ((1, 1, 1), "bf16", "whole", 1, S, False),    # pitches of one element
    ((1, 1, 1), "f32", "whole", 1, T, False),
    ((5, 70, 3), "bf16", "whole", 1, S, False),   # B rows of 6 bytes: a chunk spans rows
    ((32, 64, 128), "bf16", "whole", 8, S, False),   # one tile and one step exactly
    ((33, 65, 129), "bf16", "whole", 1, S, False),   # one more of everything
    ((31, 63, 127), "bf16", "blocks", 8, S, False),
    ((32, 32, 32), "f32", "whole", 1, T, False),
    ((33, 129, 31), "f32", "blocks", 4, T, False),
    ((65, 33, 65), "f32", "uneven", 1, T, True),
    ((300, 143, 384), "f32", "blocks", 1, T, False),
    ((555, 717, 359), "bf16", "uneven", 1, S, True),   # K tails in eleven segments, column cuts at odd places
    ((555, 717, 359), "bf16", "uneven", 8, S, True),
    ((900, 333, 1100), "bf16", "blocks", 8, H, False),
    ((1290, 260, 1030), "bf16", "blocks", 1, B, False),
    ((128, 2285, 4192), "bf16", "column", 8, B, True),   # runs of K steps, added up by a second launch
    ((13, 3121, 4999), "bf16", "column", 1, S, True),
    ((64, 5760, 1240), "bf16", "column", 8, H, True),
    ((577, 9001, 130), "bf16", "uneven", 1, B, True),    # runs that start inside segments
    ((640, 2048, 640), "f32", "blocks", 4, F, True),
    ((201, 3001, 203), "f32", "uneven", 1, F, True),
    # every shape whose sums may run uncut, ragged at all edges and with K tails
    ((401, 325, 8753), "bf16", "whole", 1, H, False),
    ((425, 347, 8583), "bf16", "uneven", 1, H, False),
    ((1317, 2034, 120), "bf16", "blocks", 8, H, True),
    ((1553, 203, 2003), "bf16", "whole", 1, B, False),
    ((1909, 343, 1495), "bf16", "uneven", 1, B, False),
    ((1909, 343, 1495), "bf16", "uneven", 8, B, False),
    ((1669, 221, 279), "f32", "blocks", 1, F, False),
    ((217, 129, 6538), "f32", "uneven", 1, F, False),
])
@pytest.mark.parametrize("c_dtype", ["f32", "bf16"])
def test_small_products(dims, dtype, kind, ldm, tile, runs, c_dtype):
    from paper_2510_08874_amd import binding
    cfg = _cfg(dims, dtype, kind)
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, ld_multiple=ldm, c_fill=float("nan"), c_dtype=c_dtype)
    _pad_with_inf(prob)
    prob.execute()
    split = prob.plan.ran_k_split()
    assert prob.plan.small_tile() == tile and (prob.plan.last_kernels().small_runs > 1) == runs
    assert split == (runs or tile == T)                  # (the four waves of a 32 x 32 tile share its K steps)
    got = prob.c_global(0)
    for t, ld, (ti, tj) in zip(prob.C.tensors, prob.C.ld, [(i, j) for i in range(prob.C.gr) for j in range(prob.C.gc)]):
        r0, r1, c0, c1 = prob.C.bounds(ti, tj)
        if t is not None and ld > c1 - c0:
            assert torch.isnan(t[:, c1 - c0:]).all(), "padding of a C tile was written"
    A64, B64 = _to_f64(A, cfg), _to_f64(B, cfg)
    C_ref = omatmul.matmul(A, B, bf16=(dtype == "bf16"))
    if c_dtype == "f32":
        _check(got, C_ref, A64, B64, cfg, cfg["name"])
    else:
        # the fp32 sum's bound, and one rounding to bf16 of a value within it
        bound = 4.0 * A64.shape[1] * 2.0 ** -24 * np.outer(np.linalg.norm(A64, axis=1), np.linalg.norm(B64, axis=0)) + 1e-30
        assert (np.abs(got.astype(np.float64) - C_ref) <= bound + (np.abs(C_ref) + bound) * 2.0 ** -8).all()
    prob.execute()
    assert np.array_equal(got, prob.c_global(0))
    prob.execute(flags=binding.DMM_NO_MERGE | (binding.DMM_C_BF16 if c_dtype == "bf16" else 0))
    assert prob.plan.small_tile() is None
    if not split:
        assert not prob.plan.ran_k_split()
        assert np.array_equal(got, prob.c_global(0))
    prob.close()
