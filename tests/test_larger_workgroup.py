"""Small-factor instances with large tiles are compiled with two workgroup sizes; long tiles take the larger one."""
import numpy as np
import pytest

import kron_inputs
import paper_2401_10187_amd as km

CASES = [("float32", 40, 5, 8, 640), ("float32", 31, 3, 12, 768), ("float32", 40, 3, 11, 768), ("float64", 60, 3, 10, 768)]


def test_long_tiles_take_the_larger_workgroup_and_short_ones_do_not():
    for dtype, M, P, N, threads in CASES:
        assert threads in [s["block"] for s in km.plan(M, [P] * N, [P] * N, dtype)], (dtype, P, N)
    for dtype, M, P, N in (("float32", 1024, 3, 7), ("float32", 1000, 5, 4), ("float64", 1000, 3, 6)):
        assert all(s["block"] == 256 for s in km.plan(M, [P] * N, [P] * N, dtype)), (dtype, P, N)


def test_a_launch_that_only_the_small_workgroup_can_make_is_still_planned():
    """A launch holds fewer than 2^32 work-items: 275114 x 5^8 is 6.9 million tiles, too many for 640 threads each."""
    for dtype, M, P, N in (("float32", 275114, 5, 8), ("float32", 1400112, 5, 7)):
        steps = km.plan(M, [P] * N, [P] * N, dtype)
        assert all(s["grid"] * s["block"] < 2 ** 32 for s in steps), (M, P, N)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,P,N,threads", CASES, ids=str)
def test_matches_the_reference(dtype, M, P, N, threads):
    """1e-5 (fp32), 1e-12 (fp64) of the largest value: sums of P terms per factor are off by at most (P + 1) N u of
    the product of absolute values."""
    import oracle
    torch = pytest.importorskip("torch")
    X, Fs = kron_inputs.make_problem(M, [(P, P)] * N, dtype, "uniform", "normal", seed=66)
    print("larger workgroup %s M=%d %d^%d" % (dtype, M, P, N), flush=True)
    got = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]).cpu().numpy()
    ref = oracle.kron_matmul(X, Fs)
    assert np.abs(got - ref).max() <= (1e-5 if dtype == "float32" else 1e-12) * np.abs(ref).max()
