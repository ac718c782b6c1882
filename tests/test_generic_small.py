"""The generic kernel's form for small factors: slices read by a thread each (P up to 8), or copied to LDS whole."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402


@pytest.fixture
def generic_only():
    old = km.get_option(km.KM_OPT_KERNELS)
    km.set_option(km.KM_OPT_KERNELS, 1)
    yield
    km.set_option(km.KM_OPT_KERNELS, old)


# (rows, factors): every number of columns per thread with columns that it divides and does not, more than one group of 32;
# slices of 1 to 9 elements, odd and even, of LDS rows at the limit and beyond it (the other form); rows of one
# slice, of fewer than a unit's 128, of just as many, of more; ragged last units
SHAPES = [(P, Q) for P in (1, 2, 3, 4, 5, 7, 8, 9, 12) for Q in (1, 2, 3, 5, 8, 9, 16, 17, 32, 33, 40)] + \
         [(64, 3), (65, 7), (127, 2), (128, 17), (129, 5), (31, 70), (100, 1)]


def _check(dtype, M, shapes, workspace=False):
    import oracle
    tol = 1e-5 if dtype == "float32" else 1e-12
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=86, **kinds)
        print("generic small %s M=%d %s" % (dtype, M, shapes), flush=True)
        n = M * int(np.prod([q for _, q in shapes]))
        frame = torch.full((n + 64,), -7.0, dtype=torch.float32 if dtype == "float32" else torch.float64, device="cuda")
        Y = frame[32:32 + n].view(M, -1)
        need = km.workspace_size(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)
        ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda") if workspace else None
        km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs], Y=Y, workspace=ws)
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        assert (frame[:32] == -7).all() and (frame[32 + n:] == -7).all()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_every_form_matches_the_reference(generic_only, dtype):
    """1e-5 (fp32), 1e-12 (fp64) of the largest value: a sum of P terms is off by at most P u of the product of absolute
    values; bit for bit on small integers; nothing is written outside Y."""
    for P, Q in SHAPES:
        assert [s["kernel"] for s in km.plan(300, [P], [Q], dtype)] == [km.KM_KERNEL_GENERIC]
        _check(dtype, 300, [(P, Q)])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("M,shapes", [(3, [(43, 2), (3, 5)]), (7, [(128, 1), (4, 4)]), (1, [(1, 1), (5, 3)]), (150, [(2, 2), (5, 40)]), (40, [(7, 2), (5, 17)]), (40, [(8, 2), (5, 17)]), (9, [(200, 1), (7, 33)]),
                                      (5, [(2, 2), (3, 4), (12, 3)]), (1100, [(3, 3), (7, 3)])], ids=str)
def test_rows_of_any_number_of_slices(generic_only, dtype, M, shapes):
    _check(dtype, M, shapes)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P", [("float32", 3), ("float32", 13), ("float64", 6), ("float64", 9)])
def test_what_is_not_finite_stays_in_its_slice(generic_only, dtype, P):
    M = 261                                                # two units and five slices
    X, Fs = kron_inputs.make_problem(M, [(P, 5)], dtype, "uniform", "normal", seed=87)
    F = [torch.from_numpy(Fs[0]).cuda()]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    X[0, 0], X[M - 1, P - 1], X[130, 0] = np.nan, np.inf, np.inf
    got = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    rest = [r for r in range(M) if r not in (0, 130, M - 1)]
    assert torch.equal(got[rest], clean[rest]) and not torch.isfinite(got[[0, 130, M - 1]]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes,tiled", [(9363, [(74, 14), (18, 5)], True), (1254, [(7, 2), (51, 23)], True),
                                            (1, [(5, 5), (5, 5), (5, 5), (2, 2)], False), (256, [(7, 2), (51, 23)], False)], ids=str)
@pytest.mark.parametrize("lanes", [True, False], ids=["as planned", "without a slice per lane"])
def test_small_mixed_problems_of_many_rows_are_tiled(M, shapes, tiled, lanes):
    """Where whole rows on the FMA kernel are the slower plan, the intermediates of the tiled launches fit the static array all the
    same.  (Those launches run in calls that bring the workspace.)  Some of them run with a slice per lane (variant -8); an option that asks for
    a workgroup size no kernel has leaves those to the generic kernel."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    old = km.get_option(km.KM_OPT_PREFER_THREADS)
    try:
        if not lanes:
            km.set_option(km.KM_OPT_PREFER_THREADS, 1)
        steps = km.plan(M, P, Q, "float32")
        assert ([s["kernel"] for s in steps] == [km.KM_KERNEL_ROWS]) != tiled
        if tiled:
            assert any(s["variant"] == -8 for s in steps) == (lanes and M == 9363)
            assert any(s["kernel"] == km.KM_KERNEL_GENERIC for s in steps) == (not lanes or M == 1254)
        assert km.workspace_size(M, P, Q, "float32") <= (km.KM_STATIC_SCRATCH_BYTES if tiled else 0)
        _check("float32", M, shapes, workspace=True)
    finally:
        km.set_option(km.KM_OPT_PREFER_THREADS, old)
