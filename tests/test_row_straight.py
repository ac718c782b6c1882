"""The whole-row kernel on the matrix cores: last steps whose results go straight to Y and those that leave through LDS."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

# four wavefronts: result rows of 8192 bytes (straight) and of the next length (in vectors, and of odd length element by element);
# sixteen: long rows, straight; contractions of one chunk, several, and a second round; wavefronts without a unit in one of the steps
CASES = [
    ("float32", 1000, [(12, 32), (12, 64)], 256), ("float32", 1000, [(12, 41), (12, 50)], 256), ("float32", 1000, [(12, 33), (12, 63)], 256),
    ("float64", 900, [(12, 16), (12, 64)], 256), ("float64", 900, [(12, 25), (12, 41)], 256),
    ("float32", 40, [(20, 60), (20, 61)], 1024), ("float64", 30, [(9, 30), (11, 43)], 1024), ("float32", 7, [(3, 2), (97, 33)], 1024),
    ("float64", 5, [(81, 17), (2, 1)], 1024), ("float32", 9, [(1, 5), (128, 1), (2, 40)], 1024),
]


@pytest.mark.parametrize("dtype,M,shapes,threads", CASES, ids=str)
def test_the_list_takes_the_kernel(dtype, M, shapes, threads):
    steps = km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)
    assert [(s["variant"], s["block"]) for s in steps] == [(-2, threads)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes,threads", CASES, ids=str)
def test_matches_the_reference(dtype, M, shapes, threads):
    """Relative to the largest value 1e-5 in fp32 and 1e-12 in fp64 (a chain of dot products of lengths P_i is off by at most
    (sum P_i + N) u of the product of absolute values); bit for bit on small integers."""
    import oracle
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=75, **kinds)
        print("row_straight %s M=%d %s" % (dtype, M, shapes), flush=True)
        got = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]).cpu().numpy()
        ref = oracle.kron_matmul(X, Fs)
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= (1e-5 if dtype == "float32" else 1e-12) * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes", [("float32", 40, [(21, 60), (18, 61)]), ("float64", 900, [(13, 25), (11, 41)])], ids=str)
def test_infinities_stay_in_their_row(dtype, M, shapes):
    """An infinity in the last element of a row, next to what a short first chunk reads past: the row's results are infinities or NaN,
    its neighbours are untouched."""
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=76)
    F = [torch.from_numpy(f).cuda() for f in Fs]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    X[5, -1] = X[M - 1, 0] = np.inf
    got = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    rest = [r for r in range(M) if r not in (5, M - 1)]
    assert torch.equal(got[rest], clean[rest])
    assert not torch.isfinite(got[5]).any() and not torch.isfinite(got[M - 1]).any()
