"""The run-time-shape MFMA kernel with the factor in registers (plan steps of that family with variant -3)."""
import numpy as np
import pytest

import kron_inputs
import paper_2401_10187_amd as km

PAD = -3


def _plan(dtype, M, shapes):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


# (dtype, rows, factors): contractions at the ends of the compiled classes (32, 64, 96, 128), slices that are whole
# 16-byte vectors and not, one to eight column blocks, rows shorter than a tile, of one slice and longer, ragged ends
CASES = [
    ("float32", 1300, [(20, 20)] * 3), ("float32", 30001, [(31, 17)]), ("float32", 3000, [(32, 8), (33, 33)]),
    ("float32", 1100, [(60, 64), (64, 63)]), ("float32", 9, [(65, 65)] * 2 + [(13, 13)]), ("float32", 1050, [(96, 80), (40, 96)]),
    ("float32", 1030, [(97, 97), (9, 13)]), ("float32", 6, [(127, 128), (128, 127), (2, 2)]), ("float32", 5, [(100, 100)] * 3),
    ("float32", 70001, [(20, 15)]), ("float32", 333, [(128, 113)]), ("float32", 1100, [(50, 33), (22, 28)]),
    ("float64", 1300, [(20, 20)] * 3), ("float64", 1111, [(31, 33), (32, 17), (16, 17)]), ("float64", 1025, [(33, 33)] * 2),
    ("float64", 1030, [(64, 48), (45, 63)]), ("float64", 40, [(96, 65), (66, 96)]), ("float64", 40, [(97, 100), (100, 113)]),
    ("float64", 4, [(128, 127), (127, 128), (3, 3)]), ("float64", 50001, [(14, 15)]), ("float64", 3, [(100, 100)] * 2 + [(7, 7)]),
]


def test_the_list_takes_the_kernel_and_its_launches_fit():
    """Grids are whole eighths (one part of the tiles per XCD), workgroups at most 1024 threads, LDS at most 96 KB."""
    for dtype, M, shapes in CASES:
        steps = [s for s in _plan(dtype, M, shapes) if s["variant"] == PAD]
        assert steps, (dtype, M, shapes)
        for s in steps:
            assert s["kernel"] == km.KM_KERNEL_MFMA_ANY and s["num_factors"] == 1
            assert s["grid"] % 8 == 0 and s["grid"] > 0 and s["block"] <= 1024 and s["lds_bytes"] <= 96 * 1024


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_matches_the_reference(dtype, M, shapes):
    """Relative to the largest value 1e-5 in fp32 and 1e-12 in fp64 (a chain of dot products of lengths P_i is off by
    at most (sum P_i + N) u of the product of absolute values); bit for bit on small integers."""
    import oracle
    torch = pytest.importorskip("torch")
    tol = 1e-5 if dtype == "float32" else 1e-12
    exact_too = 2.0 * np.prod([p for p, _ in shapes], dtype=np.float64) < (2 ** 24 if dtype == "float32" else 2 ** 53)
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        if exact and not exact_too:
            continue
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=63, **kinds)
        print("mfma_pad %s M=%d %s" % (dtype, M, shapes), flush=True)
        Y = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs])
        torch.cuda.synchronize()
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P", [("float32", 21), ("float32", 50), ("float64", 33), ("float64", 97)])
def test_nothing_leaks_between_slices(dtype, P):
    """A contraction length that is no multiple of 4 reads past its slice: an infinity there must not turn a
    neighbour into NaN, and what the last, ragged tile holds past the end must not either."""
    torch = pytest.importorskip("torch")
    M = 1027
    X, Fs = kron_inputs.make_problem(M, [(P, P)], dtype, seed=64)
    assert _plan(dtype, M, [(P, P)])[0]["variant"] == PAD
    F = [torch.from_numpy(Fs[0]).cuda()]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    X[7, 0] = X[M - 1, P - 1] = np.inf
    got = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    rest = [r for r in range(M) if r not in (7, M - 1)]
    assert torch.equal(got[rest], clean[rest])
    assert torch.isinf(got[7]).all() and torch.isinf(got[M - 1]).all()
