"""GPU parity of the kernel that takes fp32 operands apart into three bf16 each (tiles of 128 x 128), where its loop
and its way out change form: K tails, rows shorter than a chunk, tiles across the cuts of C, K dealt to several
workgroups.  Against the fp64 oracle (element bound of test_gpu_parity), and no further from it than sums of exact
products in fp32, two terms at a time; also where all terms have one sign, so that what the split leaves out adds up,
and where a sum has so few terms that the error of a product shows.
Tiles that cannot be split (infinities, NaN, values with bits below the smallest bf16) are multiplied in fp32."""
import numpy as np
import pytest

from oracle import matmul as omatmul
from tests.test_gpu_parity import _check, _device_problem
from tests.test_gpu_ring import _problem
from tests.test_gpu_small import _pad_with_inf
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pair(cfg, A, B, ldm):
    """C by the split kernel and by the macro-tiles."""
    from paper_2510_08874_amd import binding
    prob = _device_problem(cfg, A, B, ld_multiple=ldm, c_fill=float("nan"))
    _pad_with_inf(prob)
    prob.execute()
    assert prob.plan.small_tile() == (128, 128) and prob.plan.ran_k_split()
    got = prob.c_global(0)
    prob.execute(flags=binding.DMM_NO_MERGE)
    assert prob.plan.small_tile() is None
    want = prob.c_global(0)
    prob.close()
    return got, want


def _fp32_chain(A, B):
    acc = np.zeros((A.shape[0], B.shape[1]), np.float32)
    A, B = A.astype(np.float64), B.astype(np.float64)
    for k in range(0, A.shape[1], 2):
        acc = (acc + A[:, k:k + 2] @ B[k:k + 2]).astype(np.float32)
    return acc


SHAPES = [
    (2048, 1024, 2048, 1024, 1024, 2048, 2048),  # whole tiles
    (1665, 1290, 1667, 129, 1290, 1665, 1667),   # K tails of one element, one row and three columns over
    (1030, 2003, 2044, 668, 501, 515, 511),       # tiles across C's cuts, other cuts in A and B
    (1100, 4000, 1200, 4000, 18, 1100, 1200),    # segments shorter than a step
    (1790, 2050, 1917, 2050, 2050, 1790, 1917),  # odd pitches
]


@pytest.mark.parametrize("ldm", [1, 8])
@pytest.mark.parametrize("dims", SHAPES)
def test_split(dims, ldm):
    cfg = dict(_problem(*dims), dtype="f32")
    A, B = workloads.make_operands(cfg)
    for one_sign in (False, True):
        if one_sign:
            A, B = np.abs(A), np.abs(B)
        got, _ = _pair(cfg, A, B, ldm)
        ref = omatmul.matmul(A, B, bf16=False)
        _check(got, ref, A.astype(np.float64), B.astype(np.float64), cfg, cfg["name"])
        rows, cols = slice(64, 256), slice(-192, None)
        chain = _fp32_chain(A[rows], B[:, cols])
        assert np.linalg.norm((got - ref)[rows, cols]) <= np.linalg.norm(chain - ref[rows, cols])


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3e38, 3.4028235e38, 1e-37, 1.5e-45])
@pytest.mark.parametrize("dims", SHAPES[:1] + SHAPES[2:4])
def test_values_that_cannot_be_split(dims, value):
    """One such element in A and one in B: everything they do not reach as before, and what they reach as
    the macro-tiles give it.  (3e38 can be split; its products overflow, or do not.  The largest value rounds to infinity.)"""
    cfg = dict(_problem(*dims), dtype="f32")
    A, B = workloads.make_operands(cfg)
    M, K, N = dims[:3]
    A[M - 1, K - 1] = A[70, 3] = value
    B[K // 2, N - 2] = value
    got, want = _pair(cfg, A, B, 1)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    assert np.array_equal(got[np.isinf(got)], want[np.isinf(want)])
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    ok_row, ok_col = (np.abs(A64) < 1e30).all(1), (np.abs(B64) < 1e30).all(0)
    _check(got[ok_row][:, ok_col], A64[ok_row] @ B64[:, ok_col], A64[ok_row], B64[:, ok_col], cfg, cfg["name"])


# significands whose second and third parts are as large as they get: cut off after 8 bits, rounded to 8 bits
CUT = [1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -6 - 2.0 ** -22 - 2.0 ** -23]
ROUNDED = [1 + 2.0 ** -8 - 2.0 ** -16 - 2.0 ** -17 + 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -23, 1 + 2.0 ** -8 + 2.0 ** -16 + 2.0 ** -17 - 2.0 ** -23]


@pytest.mark.parametrize("values", [None, CUT, ROUNDED])
@pytest.mark.parametrize("terms", [1, 2, 8])
def test_few_terms(terms, values):
    """Rows of A with so many elements that are not zero: products are as good as exact, so that a sum has an error of
    2^-24 of it for every term.  (With more than one: what eight products of a step lose in being aligned to the largest of
    them, 2^-23 of it each, on top.)  What is left out of a product is 2^-32 of it and less."""
    cfg = dict(_problem(*SHAPES[0]), dtype="f32")
    A, B = workloads.make_operands(cfg)
    rng = np.random.default_rng(terms)
    if values:
        A, B = (np.copysign(rng.choice(np.array(values, np.float32), X.shape), X) for X in (A, B))
    kept = np.zeros(A.shape, bool)
    kept[np.arange(A.shape[0])[:, None], rng.permuted(np.tile(np.arange(A.shape[1]), (A.shape[0], 1)), axis=1)[:, :terms]] = True
    A = np.ascontiguousarray(np.where(kept, A, 0).astype(np.float32))
    got, _ = _pair(cfg, A, np.ascontiguousarray(B), 1)
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    ref = A64 @ B64
    units = terms + (2 * (terms - 1) if terms > 1 else 0)
    assert (np.abs(got - ref) <= units * 2.0 ** -24 * (1 + 2.0 ** -6) * (np.abs(A64) @ np.abs(B64))).all()


def test_long_sums_of_one_sign():
    """Operands of one sign and a long sum in one piece: nothing small is missing from it."""
    dims = (4096, 4096, 4096, 4096, 4096, 4096, 4096)
    cfg = dict(_problem(*dims), dtype="f32")
    A, B = (np.abs(X) for X in workloads.make_operands(cfg))
    got, want = _pair(cfg, A, B, 1)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.linalg.norm(got - ref) <= np.linalg.norm(want - ref)


@pytest.mark.parametrize("dims", [(1030, 2003, 2046, 668, 501, 515, 511), (1665, 1290, 1667, 129, 1290, 1665, 1667)])
def test_padding_does_not_show_in_the_bits(dims):
    """Rows whose last chunk reaches into their padding: whatever lies there (zeros, bits below the smallest bf16,
    NaN with every bit set, infinities), C has the same bits."""
    cfg = dict(_problem(*dims), dtype="f32")
    A, B = workloads.make_operands(cfg)
    prob = _device_problem(cfg, A, B, ld_multiple=8, c_fill=float("nan"))
    seen = []
    for bits in (0, 1, -1, 0x7F800000):
        for ts in (prob.A, prob.B):
            for i, t in enumerate(ts.tensors):
                _, _, c0, c1 = ts.bounds(*divmod(i, ts.gc))
                t.view(torch.int32)[:, c1 - c0:] = bits
        assert all(t.shape[1] > dims[2] for t in prob.B.tensors) and dims[2] % 4
        prob.execute()
        assert prob.plan.small_tile() == (128, 128)
        seen.append(prob.c_global(0))
    prob.close()
    for other in seen[1:]:
        assert np.array_equal(seen[0].view(np.int32), other.view(np.int32))


def test_tiny_operands():
    """Operands all below 2^-110, the other side large: as accurate as elsewhere."""
    cfg = dict(_problem(*SHAPES[2]), dtype="f32")
    A, B = workloads.make_operands(cfg)
    A, B = A * np.float32(2.0 ** -118), B * np.float32(2.0 ** 100)
    got, _ = _pair(cfg, A, B, 8)
    ref = omatmul.matmul(A, B, bf16=False)
    bound = 4.0 * SHAPES[2][1] * 2.0 ** -24 * np.outer(np.linalg.norm(A.astype(np.float64), axis=1), np.linalg.norm(B.astype(np.float64), axis=0))
    assert np.max(np.abs(got - ref) / bound) <= 1.0
