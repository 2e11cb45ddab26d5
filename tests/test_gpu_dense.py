"""GPU parity of large bf16 products whose operands are copied to dense aligned rows first (rows
that are not 16-byte aligned, many K-segments): against the fp64 oracle with the element bound of
test_gpu_parity.  Odd sizes, column cuts inside 16-byte chunks, a share of K per replica of C, and
operands in new places and with new values under one plan (nothing of the copy may be kept)."""
import numpy as np
import pytest

import workloads
from oracle import matmul as omatmul
from tests.test_gpu_parity import _check, _device_problem, _to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cyclic(M, K, N, nb, c):
    return dict(name=f"dense-bc{nb}-c{c}@{M}x{K}x{N}", M=M, K=K, N=N, dtype="bf16", nranks=8 * c,
                A=workloads.block_cyclic_desc(M, K, nb, nb, 2, 4, c), B=workloads.block_cyclic_desc(K, N, nb, nb, 2, 4, c),
                C=workloads.block_cyclic_desc(M, N, nb, nb, 2, 4, c), dist=("normal", 1.0), seeds=(61, 62))


def _uneven(M, K, N, s):
    cuts = workloads.jittered_cuts
    return dict(name=f"dense-uneven@{M}x{K}x{N}", M=M, K=K, N=N, dtype="bf16", nranks=15,
                A=workloads.desc(M, K, cuts(M, 3, s), cuts(K, 5, s + 1), 3, 5), B=workloads.desc(K, N, cuts(K, 7, s + 2), [0, N], 7, 1),
                C=workloads.desc(M, N, cuts(M, 5, s + 3), cuts(N, 3, s + 4), 5, 3), dist=("uniform", 1.0), seeds=(63, 64))


CASES = [_cyclic(4101, 2051, 4099, 100, 1), _cyclic(3001, 4099, 4102, 99, 2), _uneven(8025, 2369, 4107, 77)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c["name"])
def test_products_on_dense_copies(cfg):
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, c_fill=float("nan"))
    prob.execute()
    got = prob.c_global(0)
    A64, B64 = _to_f64(A, cfg), _to_f64(B, cfg)
    _check(got, omatmul.matmul(A, B, bf16=True), A64, B64, cfg, cfg["name"])
    prob.execute()                                       # the tables of the call before, the copy made anew
    assert np.array_equal(got, prob.c_global(0))
    for t in prob.A.tensors:                             # new values in the same place
        if t is not None:
            t.mul_(2.0)
    prob.execute()
    assert np.array_equal(2.0 * got, prob.c_global(0))   # (a power of two scales every sum exactly)
    moved = [None if t is None else t.clone() for t in prob.A.tensors]
    prob.A.tensors[:] = moved                            # the same values in new places
    prob.args = prob.plan.marshal(prob.A.tensors, prob.A.ld, prob.B.tensors, prob.B.ld, prob.C.tensors, prob.C.ld)
    prob.execute()
    assert np.array_equal(2.0 * got, prob.c_global(0))
    prob.close()
